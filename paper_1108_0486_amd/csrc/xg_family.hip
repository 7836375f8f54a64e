// HIP kernels of libxg for two further xorgens members, both with r = 64 and
// s = 33 (Section 2: s = r/2 + 1, gcd(r, s) = 1; Section 1.5: period
// 2^n - 1 for n = r w a power of two up to 4096):
//   n2048: w = 32, (a, b, c, d) = (19, 19,  9, 18), gamma = 16;
//   w64:   w = 64, (a, b, c, d) = (24, 22, 37, 45), gamma = 32;
// with x_i = x_{i-64} (I + L^a)(I + R^b) xor x_{i-33} (I + L^c)(I + R^d), the
// Weyl sequence W_k = W_{k-1} + omega (omega the odd integer nearest
// 2^{w-1}(sqrt 5 - 1)) and out_k = x_k + (W_k xor (W_k >> gamma)) mod 2^w
// (Eq. (1)).  The paper gives no shifts for these members; each quadruple
// makes the characteristic polynomial primitive of degree n.
//
// Parallel step: x_p .. x_{p+31} depend only on words older than x_p while
// 32 <= s, so a step computes 32 words of a stream.  A 64-lane wavefront runs
// two streams with interleaved lanes: lane 2j + h holds word j of stream h
// (h = 0, 1), so every lane works and a step writes 64 words.  For the chunk
// at p, lane 2j + h holds
//   prev = x_{p-64+j},  cur = x_{p-32+j}          (of stream h)
// and x_{p+j} = A(prev) xor B(x_{p+j-33}), where x_{p+j-33} is cur[j-1] for
// j >= 1 and prev[31] for j = 0.  Rotating B(cur) up by two lanes moves word
// j - 1 of each stream to word j of the same stream; lanes 0 and 1 receive
// word 31 of their own stream, which is B(prev[31]) one step later, so they
// keep the previous step's rotation (as the one-stream kernel does on lane 0).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "xg_device.h"
#include "xg_jump_mm.h"
#include "xg_normal.h"
#include "xg_normal_f64.h"
#include "xg_internal.h"
#include "xg_launch.h"
#include "xg_fam_batch.h"
#include "xg_pairs.h"

namespace xg {
namespace {

struct MemberN2048 {
  using word = uint32_t;
  static constexpr uint32_t a = 19, b = 19, c = 9, d = 18, gamma = 16;
  static constexpr word omega = 0x9E3779B9u;
  // ring u32[64] | W | reserved | pos u64
  static constexpr uint32_t state_bytes = 272, weyl_off = 256, pos_off = 264;
};

struct MemberW64 {
  using word = uint64_t;
  static constexpr uint32_t a = 24, b = 22, c = 37, d = 45, gamma = 32;
  static constexpr word omega = 0x9E3779B97F4A7C15ull;
  // ring u64[64] | W | pos
  static constexpr uint32_t state_bytes = 528, weyl_off = 512, pos_off = 520;
};

constexpr uint32_t kStep = 32;  // words of one stream per wavefront step

using dev::splitmix64_at;
using dev::xcd_block;

// Lane l receives lane l-2's value (mod 64): two one-lane rotations.
__device__ __forceinline__ uint32_t rot2(uint32_t v) { return dev::lanes_rotate_up(dev::lanes_rotate_up(v)); }
__device__ __forceinline__ uint64_t rot2(uint64_t v) {
  return (uint64_t)rot2((uint32_t)v) | ((uint64_t)rot2((uint32_t)(v >> 32)) << 32);
}

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return dev::xor3(a, b, c); }
__device__ __forceinline__ uint64_t xor3(uint64_t a, uint64_t b, uint64_t c) {
  return (uint64_t)dev::xor3((uint32_t)a, (uint32_t)b, (uint32_t)c) |
         ((uint64_t)dev::xor3((uint32_t)(a >> 32), (uint32_t)(b >> 32), (uint32_t)(c >> 32)) << 32);
}

__device__ __forceinline__ uint32_t shfl_word(uint32_t v, int src) { return (uint32_t)__shfl((int)v, src); }
__device__ __forceinline__ uint64_t shfl_word(uint64_t v, int src) {
  return (uint64_t)(uint32_t)__shfl((int)(uint32_t)v, src) |
         ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(v >> 32), src) << 32);
}

template <class M>
__device__ __forceinline__ typename M::word op_b(typename M::word v) {
  v ^= v << M::c;
  return v ^ (v >> M::d);
}

template <class M>
struct Ring2 {
  using word = typename M::word;
  word prev, cur, rprev;

  __device__ __forceinline__ void open(word p, word c) {
    prev = p;
    cur = c;
    rprev = rot2(op_b<M>(p));  // word 0: B(prev[31]) = B(x_{p-33})
  }

  // x_{p+j} on lane 2j + h; advances the ring by one chunk.
  __device__ __forceinline__ word step(bool word0) {
    const word bc = op_b<M>(cur);
    const word rc = rot2(bc);              // word j >= 1: B(x_{p+j-33}); word 0: B(x_{p-1})
    const word bs = word0 ? rprev : rc;
    const word t = prev ^ (prev << M::a);  // prev (I + L^a) (I + R^b) = t xor (t >> b)
    const word x = xor3(t, t >> M::b, bs);
    prev = cur;
    cur = x;
    rprev = rc;                            // word 0: B(x_{p-1}) = B(x_{p'-33}), p' = p + 32
    return x;
  }
};

// Output word of KIND for generator output o, as stored (FP as bit pattern).
//   w = 32: u32 o; f32 (o >> 8) 2^-24.   w = 64: u64 o; f64 (o >> 11) 2^-53.
// Both FP maps are exact (an integer of at most 24 / 53 bits times a power of 2).
template <class M, uint32_t KIND>
__device__ __forceinline__ typename M::word map_out(typename M::word o) {
  if constexpr (sizeof(typename M::word) == 4) {
    if constexpr (KIND == kU32) return o;
    else return __float_as_uint((float)(o >> 8) * 0x1p-24f);
  } else {
    if constexpr (KIND == kU64) return o;
    else return (uint64_t)__double_as_longlong((double)(o >> 11) * 0x1p-53);
  }
}

template <class M>
__device__ __forceinline__ typename M::word seed_word(uint64_t v) {
  if constexpr (sizeof(typename M::word) == 4) return (uint32_t)(v >> 32);  // the high w bits
  else return v;
}

struct Lanes {
  uint32_t lane, h, j;
  uint64_t k;    // stream index within the launch
  bool active;   // whether this half writes its stream's state
};

// The lanes of a wavefront that serves pair `pair` of a launch's `count`
// streams.  The last of an odd number of streams runs in both halves, which
// then store the same values to the same places: cheaper than a mask on every
// store of the loop.
__device__ __forceinline__ Lanes pair_lanes(uint64_t pair, uint64_t count) {
  Lanes L;
  L.lane = threadIdx.x & 63u;
  L.h = L.lane & 1u;
  L.j = L.lane >> 1;
  L.k = 2 * pair + L.h < count ? 2 * pair + L.h : count - 1;
  L.active = true;
  return L;
}

__device__ __forceinline__ uint64_t pair_of(uint32_t block) {
  return ((uint64_t)block * blockDim.x + threadIdx.x) >> 6;
}

// Writes the 64-word window that ends `rem` words into chunk x (rem in 0..31)
// as stream h's new linear ring, then W and pos.
template <class M>
__device__ __forceinline__ void store_state(unsigned char *st, const Lanes &L, typename M::word prev,
                                            typename M::word cur, typename M::word x, uint32_t rem,
                                            typename M::word weyl, uint64_t pos) {
  using word = typename M::word;
  word lo = prev, hi = cur;
  if (rem) {  // wave-uniform
    const uint32_t js = (rem + L.j) & 31u;
    const int src = (int)(2 * js + L.h);
    const word a = shfl_word(prev, src), b = shfl_word(cur, src), c = shfl_word(x, src);
    const bool wrap = rem + L.j >= 32u;
    lo = wrap ? b : a;
    hi = wrap ? c : b;
  }
  if (!L.active) return;
  word *ring = reinterpret_cast<word *>(st);
  ring[L.j] = lo;
  ring[32 + L.j] = hi;
  if (L.j == 0) {
    *reinterpret_cast<word *>(st + M::weyl_off) = weyl;
    if constexpr (sizeof(word) == 4) *reinterpret_cast<uint32_t *>(st + M::weyl_off + 4) = 0u;
    *reinterpret_cast<uint64_t *>(st + M::pos_off) = pos;
  }
}

// Seeds streams [0, num_streams): stream k from SplitMix64(seed + k) outputs
// 1 .. 64 (ring x_{-64} .. x_{-1}, high w bits) and 65 (the Weyl start); an
// all-zero ring gets x_{-1} = 1; then 4 r = 256 steps are discarded.
template <class M>
__global__ __launch_bounds__(256) void k_fam_init(unsigned char *__restrict__ state, uint64_t num_streams,
                                                  uint64_t seed) {
  using word = typename M::word;
  const uint64_t pair = pair_of(blockIdx.x);
  if (2 * pair >= num_streams) return;  // wave-uniform
  const Lanes L = pair_lanes(pair, num_streams);
  const uint64_t s = seed + L.k;
  word prev = seed_word<M>(splitmix64_at(s, L.j + 1u));
  word cur = seed_word<M>(splitmix64_at(s, L.j + 33u));
  const word w0 = seed_word<M>(splitmix64_at(s, 65u));
  const uint64_t nz = __ballot((prev | cur) != 0);
  const uint64_t mine = L.h ? 0xAAAAAAAAAAAAAAAAull : 0x5555555555555555ull;
  if ((nz & mine) == 0 && L.j == 31u) cur = 1;  // x_{-1} = 1
  Ring2<M> g;
  g.open(prev, cur);
  const bool word0 = L.j == 0;
#pragma unroll
  for (int c = 0; c < 8; ++c) (void)g.step(word0);
  store_state<M>(state + L.k * M::state_bytes, L, g.prev, g.cur, word(0), 0u, w0 + word(256) * M::omega, 0ull);
}

// A stream's state held by its half of a wavefront: ring words j and 32 + j,
// the Weyl value W_{pos-1} and the position.
template <class M>
struct FamState {
  typename M::word prev = 0, cur = 0, weyl = 0;
  uint64_t pos = 0;
};

template <class M>
__device__ __forceinline__ FamState<M> fam_load(const unsigned char *__restrict__ st, bool on, const Lanes &L) {
  using word = typename M::word;
  FamState<M> s;
  if (on) {
    const word *ring = reinterpret_cast<const word *>(st);
    s.prev = ring[L.j];
    s.cur = ring[32 + L.j];
    s.weyl = *reinterpret_cast<const word *>(st + M::weyl_off);
    s.pos = *reinterpret_cast<const uint64_t *>(st + M::pos_off);
  }
  return s;
}

// Waits here for a state's loads.  Where a use of them comes after a loop of
// stores, the wait otherwise does too, and one counter serves loads and stores
// in order, so that it waits for every store: 6 x 11422 uint32 of the 32-bit
// member 13.2 us, 12.8 with the wait in front.  THROUGH: the values pass through the
// statement, which gives the compiler's schedule of the FP64 loop 4 % (512 x
// 40001: 71.1 us and 68.3; the uint64 loop loses 1 %).  Plain launches
// only: batches gained nothing.
template <class M, bool THROUGH>
__device__ __forceinline__ void arrive(FamState<M> &s) {
  if constexpr (THROUGH) asm volatile("" : "+v"(s.prev), "+v"(s.cur), "+v"(s.weyl), "+v"(s.pos));
  else asm volatile("" : : "v"(s.prev), "v"(s.cur), "v"(s.weyl), "v"(s.pos));
}

template <bool NT, class T>
__device__ __forceinline__ void store_value(T v, T *p) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// n words of one stream per half-wavefront from state s0: the full
// steps go to o, o + stride, ... (o already offset to word j of the step),
// the ragged last step (rem = n mod 32 words) to tail + j, or after the full
// steps when tail is NULL; the end state goes to st.  on = false masks this
// lane's stores (that half's stream is absent), keep = false leaves st as it
// is; n is wave-uniform.  NT: non-temporal stores.
template <class M, uint32_t KIND, int UNROLL, bool NT = true>
__device__ __forceinline__ void fam_run(const FamState<M> &s0, unsigned char *__restrict__ st, bool on, bool keep,
                                        Lanes L, uint64_t n, typename M::word *__restrict__ o, uint64_t stride,
                                        typename M::word *__restrict__ tail) {
  using word = typename M::word;
  L.active = on && keep;
  const word w_start = s0.weyl;
  Ring2<M> g;
  g.open(s0.prev, s0.cur);
  const bool word0 = L.j == 0;
  const word wlane = word(L.j + 1u) * M::omega;  // W_{p+j} = W_{p-1} + (j + 1) omega
  word wbase = w_start;
  const uint64_t nfull = n / kStep;
  const uint32_t rem = (uint32_t)(n % kStep);
  const uint64_t nouter = nfull / UNROLL;
  for (uint64_t it = 0; it != nouter; ++it) {
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const word x = g.step(word0);
      const word w = wbase + wlane;
      wbase += word(kStep) * M::omega;
      if (on) store_value<NT>(map_out<M, KIND>(x + (word)(w ^ (w >> M::gamma))), o + u * stride);
    }
    o += UNROLL * stride;
  }
  for (uint64_t c = nouter * UNROLL; c != nfull; ++c) {
    const word x = g.step(word0);
    const word w = wbase + wlane;
    wbase += word(kStep) * M::omega;
    if (on) store_value<NT>(map_out<M, KIND>(x + (word)(w ^ (w >> M::gamma))), o);
    o += stride;
  }
  const word p0 = g.prev, c0 = g.cur;
  word x = 0;
  if (rem) {  // wave-uniform
    x = g.step(word0);
    const word w = wbase + wlane;
    word *t = tail ? tail : o;
    if (on && L.j < rem) store_value<NT>(map_out<M, KIND>(x + (word)(w ^ (w >> M::gamma))), t);
  }
  store_state<M>(st, L, p0, c0, x, rem, w_start + (word)n * M::omega, s0.pos + n);
}

// n words of each of `count` streams (launch index k = stream first + k).
// FILL = false: stream-major, out[k n + t].  FILL = true: chunk c (words
// 32c .. 32c + 31) of stream k at out[(c count + k) 32 ..], the ragged last
// chunks (rem = n mod 32 words each) packed after them at
// out[32 (n / 32) count + k rem ..]; a wavefront's step then writes 64
// adjacent words.  NT: non-temporal stores.
template <class M, uint32_t KIND, int UNROLL, bool FILL, bool NT>
__device__ __forceinline__ void fam_serve(unsigned char *__restrict__ state, const Lanes &L, uint64_t first,
                                          uint64_t count, uint64_t n, typename M::word *__restrict__ out) {
  using word = typename M::word;
  unsigned char *st = state + (first + L.k) * M::state_bytes;
  FamState<M> s0 = fam_load<M>(st, true, L);
  arrive<M, KIND == kF64>(s0);
  if constexpr (FILL) {
    word *tail = out + (n / kStep) * count * kStep + L.k * (n % kStep) + L.j;
    fam_run<M, KIND, UNROLL, NT>(s0, st, true, true, L, n, out + L.k * kStep + L.j, count * kStep, tail);
  } else {
    fam_run<M, KIND, UNROLL, NT>(s0, st, true, true, L, n, out + L.k * n + L.j, kStep, nullptr);
  }
}

// ---------------------------------------------------------------------------
// normals: Box-Muller on consecutive pairs (o_{2m}, o_{2m+1}) of each
// stream's outputs of the call, as for Section 2's member; FP32 from the
// 32-bit member, FP64 (53-bit uniforms) from the 64-bit member.  Two steps
// give 64 words of each stream, i.e. 32 pairs, one per lane: on even j words j
// and j + 1 of the first step, on odd j words j - 1 and j of the second, so
// each lane needs one word of the lane two away, which a quad permutation
// supplies in the VALU (in place of four LDS permutes per 32-bit word).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t swap_words(uint32_t v) {
  constexpr int kSwapTwo = 0x4E;  // quad_perm [2, 3, 0, 1]
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kSwapTwo, 0xF, 0xF, false);
}
__device__ __forceinline__ uint64_t swap_words(uint64_t v) {
  return (uint64_t)swap_words((uint32_t)v) | ((uint64_t)swap_words((uint32_t)(v >> 32)) << 32);
}
__device__ __forceinline__ uint32_t select_word(uint32_t a, uint32_t b, uint32_t m) { return dev::select_bits(a, b, m); }
__device__ __forceinline__ uint64_t select_word(uint64_t a, uint64_t b, uint32_t m) {
  return (uint64_t)dev::select_bits((uint32_t)a, (uint32_t)b, m) |
         ((uint64_t)dev::select_bits((uint32_t)(a >> 32), (uint32_t)(b >> 32), m) << 32);
}

// The lane's pair of the 64-word block lo | hi; its first word's place in the
// block is fam_pair_offset.  (Bit selects, not ternaries, so that the swaps
// stay outside lane-divergent code.)
template <typename word>
__device__ __forceinline__ void fam_gather_pair(word lo, word hi, uint32_t j, word &e, word &o) {
  const uint32_t odd = 0u - (j & 1u);
  const word lo_sw = swap_words(lo), hi_sw = swap_words(hi);
  e = select_word(hi_sw, lo, odd);
  o = select_word(hi, lo_sw, odd);
}
__device__ __forceinline__ uint32_t fam_pair_offset(uint32_t j) { return (j & ~1u) + ((j & 1u) << 5); }

// The normals of P pairs: in order, or (ORDERED = false) each pair's two in
// whichever order is cheaper.
struct NoConsts {};
template <bool ORDERED, int P>
__device__ __forceinline__ void fam_pairs(const NoConsts &, const uint32_t (&e)[P], const uint32_t (&o)[P],
                                          float (&z0)[P], float (&z1)[P]) {
#pragma unroll
  for (int u = 0; u < P; ++u) {
    if constexpr (ORDERED) dev::box_muller(e[u], o[u], z0[u], z1[u]);
    else dev::box_muller_unordered(e[u], o[u], z0[u], z1[u]);
  }
}
template <bool ORDERED, int P>
__device__ __forceinline__ void fam_pairs(const dev::ConstsF64 &k, const uint64_t (&e)[P], const uint64_t (&o)[P],
                                          double (&z0)[P], double (&z1)[P]) {
  dev::box_muller_f64<ORDERED>(k, e, o, z0, z1);
}

// Compensated FP64 sums of z and z^2 kept by one lane (one update per pair).
struct MomentsF64 {
  double s1, c1, s2, c2;
};

__device__ __forceinline__ void kahan_add_f64(double &s, double &c, double v) {
  const double y = v - c;
  const double t = s + y;
  c = (t - s) - y;
  s = t;
}

// A pair (or, has1 = false, its first variate alone) into the lane's sums, as
// z0 + z1 and fma(z1, z1, z0 z0): one compensated update each.
__device__ __forceinline__ void sums_add(dev::Moments &m, float z0, float z1) {
  dev::group_add(m, z0, z1);
  dev::group_close(m);
}
__device__ __forceinline__ void sums_add(MomentsF64 &m, double z0, double z1) {
  kahan_add_f64(m.s1, m.c1, z0 + z1);
  kahan_add_f64(m.s2, m.c2, fma(z1, z1, z0 * z0));
}

// The normals' LDS: two slots of two blocks (128 words of each stream, 32 apart
// in the banks) per wavefront.
constexpr uint32_t kFamStage = 2 * (128 + 32);
extern __shared__ __align__(16) unsigned char fam_lds[];

template <typename word>
__device__ __forceinline__ word *fam_stage() {
  return reinterpret_cast<word *>(fam_lds) + (threadIdx.x >> 6) * (2 * kFamStage);
}

template <class M>
using real_of = typename std::conditional<sizeof(typename M::word) == 8, double, float>::type;

// n normals of one stream per half-wavefront (n wave-uniform) from state s0,
// 2 ceil(n / 2) words: Box-Muller on consecutive pairs, written from o_s
// (the stream's first output) unless MOMENTS, which instead reduces the
// half's sums of z and z^2 and stores them at sums (two reals); the end state
// goes to st.  on = false masks this lane's stores, BOTH: on is true on every
// lane; keep = false leaves st as it is.  NT: non-temporal stores.
//
// The blocks wholly below n run UNROLL at a time without a test per value, and
// a pair's two adjacent stores become one (which needs the alignment of one
// value only).  One block at a time with a test per value and, for odd n, two
// separate stores per pair took 570 us for 3001 streams x 65537 FP32 normals,
// this form 235 us.
template <class M, bool MOMENTS, bool BOTH, bool NT, bool STAGED = false>
__device__ __forceinline__ void fam_normals_run(const FamState<M> &s0, unsigned char *__restrict__ st, bool on,
                                                bool keep, Lanes L, uint64_t n, real_of<M> *__restrict__ o_s,
                                                real_of<M> *__restrict__ sums) {
  using word = typename M::word;
  using real = real_of<M>;
  constexpr bool kW64 = sizeof(word) == 8;
  if constexpr (BOTH) on = true;
  L.active = on && keep;
  const word w_start = s0.weyl;
  const uint64_t pos = s0.pos;
  Ring2<M> g;
  g.open(s0.prev, s0.cur);
  const bool word0 = L.j == 0;
  const word wlane = word(L.j + 1u) * M::omega;
  word wbase = w_start;
  auto next = [&]() {
    const word x = g.step(word0);
    const word w = wbase + wlane;
    wbase += word(kStep) * M::omega;
    return word(x + (w ^ (w >> M::gamma)));
  };
  const uint64_t words = n + (n & 1u);
  const uint64_t nblk = words >> 6;  // 64-word blocks: 32 pairs of each stream
  const uint64_t nsafe = n >> 6;     // of these, the blocks whose 64 normals are all below n
  const uint32_t rw = (uint32_t)(words & 63u);
  const uint32_t poff = fam_pair_offset(L.j);
  constexpr int UNROLL = kW64 ? 2 : 4;
  static_assert(!(STAGED && kW64), "the staged gather is the 32-bit member's");
  typename std::conditional<kW64, MomentsF64, dev::Moments>::type m;
  if constexpr (kW64) m = MomentsF64{0.0, 0.0, 0.0, 0.0};
  else m = dev::Moments{0.0f, 0.0f, 0.0f, 0.0f, -0.0f, -0.0f};
  typename std::conditional<kW64, dev::ConstsF64, NoConsts>::type consts;
  if constexpr (kW64) consts = dev::consts_f64();
  real *p = MOMENTS ? nullptr : o_s + (STAGED ? 4 * L.j : poff);
  uint64_t b = 0;
  for (const uint64_t nouter = nsafe & ~uint64_t(UNROLL - 1); b != nouter; b += UNROLL) {
    word e[UNROLL], o[UNROLL];
    real z0[UNROLL], z1[UNROLL];
    if constexpr (STAGED) {
      // Two blocks at a time through the wavefront's LDS: each lane reads four
      // consecutive words of its stream back, two pairs.
      word *stage = fam_stage<word>();
#pragma unroll
      for (int u = 0; u < UNROLL; u += 2) {
        word *half = stage + kFamStage * ((u / 2) & 1) + L.h * (128u + 32u);
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c) half[kStep * c + L.j] = next();
        dev::wave_lds_sync();  // the reads below take other lanes' words
        const word *four = half + 4 * L.j;
        e[u] = four[0];
        o[u] = four[1];
        e[u + 1] = four[2];
        o[u + 1] = four[3];
        dev::wave_lds_sync();  // the next writes to this half come after these reads
      }
    } else {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        const word oa = next();
        const word ob = next();
        fam_gather_pair(oa, ob, L.j, e[u], o[u]);
      }
    }
    fam_pairs<!MOMENTS>(consts, e, o, z0, z1);
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      if constexpr (!MOMENTS) {
        real *q = STAGED ? p + 128 * (u / 2) + 2 * (u % 2) : p + 64 * u;
        if (on) {
          store_value<NT>(z0[u], q);
          store_value<NT>(z1[u], q + 1);
        }
      } else if constexpr (kW64) {
        sums_add(m, z0[u], z1[u]);
      } else {
        dev::group_add(m, z0[u], z1[u]);
      }
    }
    if constexpr (MOMENTS && !kW64) dev::group_close(m);  // one compensated update per UNROLL pairs
    if constexpr (!MOMENTS) p += 64 * UNROLL;
  }
  // Pair at idx, idx + 1 of the call, those below n.
  auto checked = [&](word e, word o, uint64_t idx) {
    const word ee[1] = {e}, oo[1] = {o};
    real y0[1], y1[1];
    fam_pairs<true>(consts, ee, oo, y0, y1);
    const real z0 = y0[0], z1 = y1[0];
    const bool has0 = on && idx < n, has1 = on && idx + 1 < n;
    if constexpr (MOMENTS) {
      if (has0) sums_add(m, z0, has1 ? z1 : real(0));  // has1 implies has0
    } else {
      if (has0) store_value<NT>(z0, o_s + idx);
      if (has1) store_value<NT>(z1, o_s + idx + 1);
    }
  };
  for (; b != nblk; ++b) {
    const word oa = next();
    const word ob = next();
    word e, o;
    fam_gather_pair(oa, ob, L.j, e, o);
    checked(e, o, (b << 6) + poff);
  }
  // Tail: rw (even, < 64) more words.
  word p0 = g.prev, c0 = g.cur, xl = 0;
  uint32_t rem = 0u;
  if (rw) {  // wave-uniform
    word oa, ob = 0;
    if (rw <= 32u) {
      const word w = wbase + wlane;
      xl = g.step(word0);
      oa = xl + (w ^ (w >> M::gamma));
      rem = rw & 31u;  // rw == 32 completes the step
      if (!rem) {
        p0 = g.prev;
        c0 = g.cur;
      }
    } else {
      oa = next();
      p0 = g.prev;
      c0 = g.cur;
      const word w = wbase + wlane;
      xl = g.step(word0);
      ob = xl + (w ^ (w >> M::gamma));
      rem = rw - 32u;
    }
    word e, o;
    fam_gather_pair(oa, ob, L.j, e, o);
    if (poff < rw) checked(e, o, (nblk << 6) + poff);
  }
  store_state<M>(st, L, p0, c0, xl, rem, w_start + (word)words * M::omega, pos + words);
  if constexpr (MOMENTS) {
    // Folded and reduced across the stream's lanes in FP64 (for the FP32
    // sums: rounded once to FP32 at the end).
    double v1 = (double)m.s1 - (double)m.c1, v2 = (double)m.s2 - (double)m.c2;
#pragma unroll
    for (int off = 32; off >= 2; off >>= 1) {  // even offsets keep each stream's lanes apart
      v1 += __shfl_xor(v1, off);
      v2 += __shfl_xor(v2, off);
    }
    if (on && L.j == 0) {
      sums[0] = (real)v1;
      sums[1] = (real)v2;
    }
  }
}

// n normals of each of `count` streams (launch index k = stream first + k)
// at out[k n + t], or their sums at sums[2k], sums[2k + 1].  Consumes
// 2 ceil(n / 2) words per stream.
template <class M, bool MOMENTS, bool NT, bool STAGED>
__global__ __launch_bounds__(1024) void k_fam_normals(unsigned char *__restrict__ state, uint64_t first,
                                                      uint64_t count, uint64_t n, void *__restrict__ out_v,
                                                      void *__restrict__ sums_v) {
  using real = real_of<M>;
  const uint64_t pair = pair_of(xcd_block());
  if (2 * pair >= count) return;  // wave-uniform
  const Lanes L = pair_lanes(pair, count);
  unsigned char *st = state + (first + L.k) * M::state_bytes;
  real *out = MOMENTS ? nullptr : static_cast<real *>(out_v) + L.k * n;
  real *sums = MOMENTS ? static_cast<real *>(sums_v) + 2 * L.k : nullptr;
  fam_normals_run<M, MOMENTS, true, NT, STAGED>(fam_load<M>(st, true, L), st, true, true, L, n, out, sums);
}

template <class M, uint32_t KIND, int UNROLL, bool FILL, bool NT>
__global__ __launch_bounds__(1024) void k_fam_generate(unsigned char *__restrict__ state, uint64_t first,
                                                       uint64_t count, uint64_t n, void *__restrict__ out) {
  // Stream-major: each XCD takes a contiguous range of streams; bulk fill:
  // plain order, so every XCD's writes spread over the whole dense front
  // (each measured the faster for its layout).
  const uint64_t pair = pair_of(FILL ? blockIdx.x : xcd_block());
  if (2 * pair >= count) return;  // wave-uniform
  fam_serve<M, KIND, UNROLL, FILL, NT>(state, pair_lanes(pair, count), first, count, n,
                                       reinterpret_cast<typename M::word *>(out));
}

// ---------------------------------------------------------------------------
// Batched requests (the persistent launch of xg_generate_batch) for these
// members.  A wavefront serves two request groups at once, one per
// half-wavefront (lanes 2j + h serve group 2p + h of pair p: first the pair
// of the wavefront's own index in the grid, then pairs taken from the atomic
// queue work[0]).  Each loop trip runs min(words left in the two
// current requests) through fam_run, with the state written back between
// trips, so both halves step together; a half whose group is done, or whose
// current request has the other output type, is masked for that trip (half
// 0 goes first).  While a half's next word falls inside a 32-word line of the
// output, a one-step head trip (fam_head) first brings each such half to its
// line's end, so that full steps store whole aligned lines.  Requests are
// uint32 / uint64 (XG_U32), FP32 / FP64 (XG_F32) or normals of that precision
// (XG_NORMAL), in elements of the member's word width; a request or group
// that fails the bounds check (stream, dtype, flags 0, output range, group
// offsets) is skipped and sets work[1].  Every wavefront exits once the queue
// passes work[2] groups.
// ---------------------------------------------------------------------------
// One generator step of the stream at st, of which this half writes the
// first `head` words (head < 32, per half; 0 writes nothing and leaves the
// state as it was) as integers or, if real, as uniform reals; the state then
// stands `head` words further on.  Branch-free in head, so every lane takes
// part in the shuffles.
template <class M, uint32_t KINT, uint32_t KREAL>
__device__ __forceinline__ void fam_head(unsigned char *__restrict__ st, bool on, const Lanes &L, uint32_t head,
                                         bool real, typename M::word *__restrict__ o) {
  using word = typename M::word;
  word *ring = reinterpret_cast<word *>(st);
  word prev = 0, cur = 0, w_start = 0;
  uint64_t pos = 0;
  if (on) {
    prev = ring[L.j];
    cur = ring[32 + L.j];
    w_start = *reinterpret_cast<const word *>(st + M::weyl_off);
    pos = *reinterpret_cast<const uint64_t *>(st + M::pos_off);
  }
  Ring2<M> g;
  g.open(prev, cur);
  const word x = g.step(L.j == 0);
  const word w = w_start + word(L.j + 1u) * M::omega;
  const word v = x + (word)(w ^ (w >> M::gamma));
  if (on && L.j < head) __builtin_nontemporal_store(real ? map_out<M, KREAL>(v) : map_out<M, KINT>(v), o);
  // The new ring: the 64-word window ending `head` words into x.
  const uint32_t js = (head + L.j) & 31u;
  const int src = (int)(2 * js + L.h);
  const word a = shfl_word(prev, src), b = shfl_word(cur, src), c = shfl_word(x, src);
  const bool wrap = head + L.j >= 32u;
  if (!on) return;
  ring[L.j] = wrap ? b : a;
  ring[32 + L.j] = wrap ? c : b;
  if (L.j == 0) {
    *reinterpret_cast<word *>(st + M::weyl_off) = w_start + (word)head * M::omega;
    *reinterpret_cast<uint64_t *>(st + M::pos_off) = pos + head;
  }
}

// Lane src's value of v, held in scalar registers.
__device__ __forceinline__ uint64_t lane_value(uint64_t v, int src) {
  const uint64_t x = shfl_word(v, src);
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32) |
         (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
}

// How evenly pairs of groups run, by up to 32 of them spread over the table and
// each group's first request.  The halves of a wavefront part where either's
// request ends, which costs a trip of the loop, and run one type at a time.
//  - apart: a wavefront for each group is faster, where there are enough: pairs
//    of two types take each other's time (384 requests of mixed types and 2^8 to 2^14
//    words on 200 streams, plan and batch in us, pairs and alone: 97 and 60, 64 bits
//    167 and 95), and pairs of two lengths more trips (lone_groups_pay).
//  - uneven: pairs of different types, or of several requests of different
//    lengths, whose times differ more than their costs.
// Types and lengths count where a quarter of the pairs differ, or where one pair
// of two types is long enough to end last.
struct PairLook {
  bool apart, uneven;
};
__device__ __forceinline__ uint32_t other_half(uint32_t v) { return dev::lane_xor<1>(v); }
__device__ __forceinline__ float other_half(float v) { return __uint_as_float(dev::lane_xor<1>(__float_as_uint(v))); }
__device__ __forceinline__ uint32_t of_lane0(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ float of_lane0(float v) { return __uint_as_float(of_lane0(__float_as_uint(v))); }

template <class M>
__device__ __forceinline__ PairLook look_at_pairs(const xg_request *__restrict__ reqs, uint32_t num_reqs,
                                                  const uint32_t *__restrict__ groups, uint32_t num_groups,
                                                  uint32_t simds, const Lanes &L) {
  uint32_t type = 0, count = 0, first = 0;
  float n = 0.0f;  // of the first request
  if (num_groups) {
    const uint32_t pairs = (uint32_t)((num_groups + 1ull) / 2);
    first = 2u * (uint32_t)((uint64_t)L.j * pairs / 32u);  // of the pair this lane and the next look at
    const uint32_t g = first + L.h < num_groups ? first + L.h : first;
    const uint32_t r = groups[g], end = groups[g + 1];
    if (r < end && r < num_reqs) {
      type = reqs[r].dtype;
      n = reqs[r].n >> 32 ? 4294967296.0f : (float)(uint32_t)reqs[r].n;
      count = end - r;
    }
  }
  constexpr int kQuarter = 16;  // lanes, two to a pair
  const float words = n * (float)count, time = type == XG_NORMAL ? 2.0f * words : words;  // of the group
  const float both = time + other_half(time);
  const uint32_t counts = count + other_half(count), more = count > counts - count ? count : counts - count;
  const bool types = other_half(type) != type, lengths = other_half(n) != n;
  // Lane 0 has the first group, and groups fall in cost.
  const bool last = __any(types && both > 1.25f * of_lane0(time)) != 0;
  const bool by_type = last || __popcll(__ballot(types)) >= kQuarter;
  // The groups around the first that share a SIMD with others.
  float second = 0.0f;
  if (num_groups > simds) {
    const uint32_t around = num_groups / 8u;
    const bool here = first + around >= simds && first <= simds + around;
    const int seen = __popcll(__ballot(here));
    second = here ? words : 0.0f;
#pragma unroll
    for (int d = 32; d; d >>= 1) second += __shfl_xor(second, d);
    second = seen ? of_lane0(second) / (float)seen : 0.0f;
  }
  const bool ends = __popcll(__ballot(types || lengths)) >= kQuarter &&
                    lone_groups_pay(sizeof(typename M::word) == 8, of_lane0(type) == XG_NORMAL, of_lane0(more),
                                    of_lane0(words), second);
  return {by_type || ends, last || __popcll(__ballot(types || (counts > 2u && lengths))) >= kQuarter};
}

template <class M, int UNROLL>
__global__ __launch_bounds__(1024) void k_fam_batch(unsigned char *__restrict__ state, uint64_t num_streams,
                                                    const xg_request *__restrict__ reqs,
                                                    const uint32_t *__restrict__ groups,
                                                    void *__restrict__ out_v, uint64_t out_elems,
                                                    uint32_t *__restrict__ work, uint32_t simds) {
  const uint32_t num_groups = work[2], num_reqs = work[3];
  using word = typename M::word;
  constexpr uint32_t kInt = sizeof(word) == 4 ? kU32 : kU64;
  constexpr uint32_t kReal = sizeof(word) == 4 ? kF32 : kF64;
  using real = typename std::conditional<sizeof(word) == 8, double, float>::type;
  word *out = reinterpret_cast<word *>(out_v);
  Lanes L;
  L.lane = threadIdx.x & 63u;
  L.h = L.lane & 1u;
  L.j = L.lane >> 1;
  L.k = 0;
  L.active = true;
  // Queue items are pairs of groups (one per half) or lone groups, largest
  // first, handed out as k_batch's: the first by the wavefront's index in the
  // grid, later ones dealt or from the counter.  Pairs that hold each other up
  // differ more in time than in cost, so fewer of them are dealt (16384 requests of
  // mixed types and 2^8 to 2^14 words: 157 us from the queue, 177 dealt; two of
  // mixed types and 2^12 words on each of 6000 streams: 126 and 137), even ones up to 64 KB
  // (two uint32 requests of 2^12 words on each: 117 and 98; 16384 of 2^8 to 2^15
  // uint64, not dealt: 255 and 269).
  constexpr uint32_t kDealEven = (1u << 16) / sizeof(word);
  const uint32_t wpb = blockDim.x >> 6;
  const uint32_t waves = gridDim.x * wpb;
  const PairLook look = look_at_pairs<M>(reqs, num_reqs, groups, num_groups, simds, L);
  const bool alone = num_groups <= waves && look.apart;
  const uint32_t num_pairs = alone ? num_groups : (uint32_t)((num_groups + 1ull) / 2);
  const uint32_t wave = blockIdx.x * wpb + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const bool dealt = alone || deal_items(reqs, num_reqs, groups, num_groups, 2 * waves, look.uneven ? 1u << 12 : kDealEven);
  uint32_t p0 = wave;
  uint32_t take = 1, round = 0;
  for (;;) {
    if (p0 >= num_pairs) break;
    const uint32_t p_end = num_pairs - p0 < take ? num_pairs : p0 + take;
    uint64_t served = 0;  // words of the trips run for these pairs
    for (uint32_t p = p0; p < p_end; ++p) {
      const uint64_t g = alone ? p : 2ull * p + L.h;  // alone: both halves run it, as a lone stream's do
      uint32_t r = 0, r_end = 0;
      if (g < num_groups) {
        r = groups[g];
        r_end = groups[g + 1];
        if (r > r_end || r_end > num_reqs) {
          if (L.j == 0) atomicOr(&work[1], 1u);
          r = r_end = 0;
        }
      }
      uint64_t done = 0;  // words of the half's current request already written
      for (;;) {
        // Each half moves past bad and empty requests (no cross-lane work here).
        xg_request q{};
        bool have = false;
        while (r < r_end) {
          q = reqs[r];
          const bool ok = q.stream < num_streams && q.dtype <= XG_NORMAL && q.flags == 0u &&
                          q.out_offset <= out_elems && q.n <= out_elems - q.out_offset;
          if (ok && q.n > done) {
            have = true;
            break;
          }
          if (!ok && L.j == 0) atomicOr(&work[1], 1u);
          ++r;
          done = 0;
        }
        const uint64_t left = have ? q.n - done : 0;
        const uint64_t left0 = lane_value(left, 0), left1 = lane_value(left, 1);
        if (left0 == 0 && left1 == 0) break;
        // Position of the half's next word within a 32-word line of the output.
        // (Normals are written pair by pair and are not realigned.)
        const uint32_t mis = have && q.dtype != XG_NORMAL
                                 ? (uint32_t)((reinterpret_cast<uintptr_t>(out) / sizeof(word) + q.out_offset + done) % kStep)
                                 : 0u;
        const uint32_t mis0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)__shfl((int)mis, 0));
        const uint32_t mis1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)__shfl((int)mis, 1));
        if (mis0 != 0u || mis1 != 0u) {
          // Head trip: one step, in which each half that starts inside a line
          // writes only up to that line's end, so its later full steps store
          // whole aligned lines (dense request offsets start most requests
          // inside a line, which measured twice as slow).
          const uint32_t head = mis != 0u ? (uint32_t)(left < kStep - mis ? left : kStep - mis) : 0u;
          const bool mine = head != 0u;
          unsigned char *st = state + (mine ? q.stream : 0) * M::state_bytes;
          word *o = out + (mine ? q.out_offset + done : 0) + L.j;
          fam_head<M, kInt, kReal>(st, mine, L, head, q.dtype == XG_F32, o);
          if (mine) {
            done += head;
            if (done == q.n) {
              ++r;
              done = 0;
            }
          }
          continue;
        }
        const uint32_t dt0 = (uint32_t)__builtin_amdgcn_readfirstlane(__shfl((int)q.dtype, 0));
        const uint32_t dt1 = (uint32_t)__builtin_amdgcn_readfirstlane(__shfl((int)q.dtype, 1));
        bool run0 = left0 != 0;
        bool run1 = left1 != 0 && (!run0 || dt0 == dt1);
        uint64_t n = run0 ? (run1 && left1 < left0 ? left1 : left0) : left1;
        const uint32_t kind = run0 ? dt0 : dt1;
        if (kind == XG_NORMAL && (n & 1u)) {
          // An odd count drops the second variate of its last pair, so only a
          // half that finishes its request with this trip may take one.
          const bool fin0 = run0 && left0 == n, fin1 = run1 && left1 == n;
          if ((run0 && !fin0) || (run1 && !fin1)) {
            if (n > 1) {
              n -= 1;
            } else {
              run0 = fin0;
              run1 = fin1;
            }
          }
        }
        const bool mine = L.h ? run1 : run0;
        unsigned char *st = state + (mine ? q.stream : 0) * M::state_bytes;
        const uint64_t at = mine ? q.out_offset + done : 0;
        if (kind == XG_NORMAL)
          fam_normals_run<M, false, false, true>(fam_load<M>(st, mine, L), st, mine, true, L, n, reinterpret_cast<real *>(out) + at, nullptr);
        else if (kind == XG_F32)
          fam_run<M, kReal, UNROLL>(fam_load<M>(st, mine, L), st, mine, true, L, n, out + at + L.j, kStep, nullptr);
        else
          fam_run<M, kInt, UNROLL>(fam_load<M>(st, mine, L), st, mine, true, L, n, out + at + L.j, kStep, nullptr);
        served += n;
        if (mine) {
          done += n;
          if (done == q.n) {
            ++r;
            done = 0;
          }
        }
      }
    }
    if (dealt) {
      p0 = dealt_item(++round, wave, waves, num_pairs);
      continue;
    }
    take = batch_take(served, p_end - p0, p0, num_pairs, waves);
    uint32_t c = 0;
    if (L.lane == 0) c = atomicAdd(&work[0], take);
    p0 = waves + (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
  }
}

template <class M>
hipError_t launch_fam_batch_k(uint32_t unroll, uint64_t blocks, dim3 block, int num_cus, unsigned char *state,
                              uint64_t num_streams, const xg_request *reqs, const uint32_t *groups, void *out,
                              uint64_t out_elems, uint32_t *work, hipStream_t stream) {
  auto run = [&](auto kernel) {
    return launch_persistent(kernel, blocks, block, 0, num_cus, stream, state, num_streams, reqs, groups, out,
                             out_elems, work, 4u * (uint32_t)(num_cus > 0 ? num_cus : 1));
  };
  switch (unroll) {
    case 1: return run(k_fam_batch<M, 1>);
    case 2: return run(k_fam_batch<M, 2>);
    case 4: return run(k_fam_batch<M, 4>);
    default: return run(k_fam_batch<M, 8>);
  }
}

// ---------------------------------------------------------------------------
// skip: advance each stream by J words without producing them.
//
// JUMP = false: the x-part steps through the J words (J small).
// JUMP = true: T^J = g(T), g = z^J mod P of degree < n (Cayley-Hamilton), is
// evaluated on the state S0 by Horner's rule in steps of 32 words:
//   S <- T^32 S  xor  sum_{i < 32} g_{32c + i} T^i S0,   c = n/32 - 1 .. 0.
// T^32 S is one generator step of the x-part.  T^i S0 is the 64-word window
// starting i words into S0's continuation E = ring | the next 32 words, so
// lane 2j + h needs E[j .. j + 63] of its stream: E is staged through LDS once
// and kept in registers.  The bits of g are wave-uniform (both streams of a
// wavefront jump by the same J).  W advances by J omega and pos by J.
// ---------------------------------------------------------------------------
template <class M, bool JUMP>
__global__ __launch_bounds__(256) void k_fam_skip(unsigned char *__restrict__ state, uint64_t first,
                                                  uint64_t count, uint64_t J, JumpPoly g) {
  using word = typename M::word;
  constexpr uint32_t kN = 64u * 8u * sizeof(word);  // n = r w with r = 64
  const uint64_t pair = pair_of(blockIdx.x);
  if (2 * pair >= count) return;  // wave-uniform
  const Lanes L = pair_lanes(pair, count);
  unsigned char *st = state + (first + L.k) * M::state_bytes;
  const FamState<M> s0 = fam_load<M>(st, true, L);
  const word prev = s0.prev, cur = s0.cur, w_start = s0.weyl;
  const uint64_t pos = s0.pos;
  const bool word0 = L.j == 0;
  const word w_end = w_start + (word)J * M::omega;
  if constexpr (!JUMP) {
    Ring2<M> r;
    r.open(prev, cur);
    const uint64_t nfull = J / kStep;
    const uint32_t rem = (uint32_t)(J % kStep);
    for (uint64_t c = 0; c != nfull; ++c) (void)r.step(word0);
    const word p0 = r.prev, c0 = r.cur;
    word x = 0;
    if (rem) x = r.step(word0);
    store_state<M>(st, L, p0, c0, x, rem, w_end, pos + J);
  } else {
    Ring2<M> r;
    r.open(prev, cur);
    const word nxt = r.step(word0);            // x_{p+j}: the continuation's next 32 words
    word *E = reinterpret_cast<word *>(fam_lds) + (threadIdx.x >> 6) * 192u + L.h * 96u;
    E[L.j] = prev;
    E[32 + L.j] = cur;
    E[64 + L.j] = nxt;
    dev::wave_lds_sync();                      // the reads below take other lanes' words
    word e[64];
#pragma unroll
    for (int i = 0; i < 64; ++i) e[i] = E[L.j + i];
    word sp = 0, sc = 0;                       // S: words j and 32 + j of the accumulated state
    for (int c = (int)(kN / kStep) - 1; c >= 0; --c) {
      if (c != (int)(kN / kStep) - 1) {
        Ring2<M> t;
        t.open(sp, sc);
        const word x = t.step(word0);
        sp = sc;
        sc = x;
      }
      const uint32_t bits = (uint32_t)(g.w[c >> 1] >> ((c & 1) * 32));
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        const word m = (word)0 - (word)((bits >> i) & 1u);
        sp ^= e[i] & m;
        sc ^= e[32 + i] & m;
      }
    }
    store_state<M>(st, L, sp, sc, word(0), 0u, w_end, pos + J);
  }
}

// ---------------------------------------------------------------------------
// Jumps on the matrix cores (xg_jump_mm.h) by a workgroup per pair of streams,
// and rows cut into parts (xg_split.h).
// ---------------------------------------------------------------------------
// r = 64 words, so the result has two tiles and the continuation n / 64 + 1
// blocks; a 64-bit word's halves are two planes of 32 bits that share G.
template <class M>
struct FamJump {
  static constexpr uint32_t kWaves = 8;
  static constexpr uint32_t kRuns = kWaves / 2;                    // wavefronts of one stream
  static constexpr uint32_t kPlanes = sizeof(typename M::word) / 4;
  static constexpr uint32_t kBits = 64 * 32 * kPlanes;             // n
  static constexpr uint32_t kBlocks = kBits / 64 + 1;
  static constexpr uint32_t kWords = kBits / 32;                   // 32-bit words of z^J mod P
  static constexpr int kQ0 = -1;                                   // G's first q (tile 1 of block 0)
  static constexpr uint32_t kQs = 2 * kBlocks - kQ0;

  struct Lds {
    uint32_t s[2][kPlanes][64 * kBlocks];     // both streams' continuations by planes
    uint32_t g[kWords];
    uint32_t rows[32 * kQs];                  // toeplitz_word(q, row_word(rho)) at 32 (q - kQ0) + rho
    uint32_t part[kWaves][kPlanes][64];       // each wavefront's share of the result
  };

  // G's rows of the polynomial g (its words in any memory).  Ends with a barrier.
  static __device__ __forceinline__ void lay_out(const uint32_t *g, Lds &lds) {
    __syncthreads();  // an earlier jump's reads of lds are done
    for (uint32_t i = threadIdx.x; i < kWords; i += 64 * kWaves) lds.g[i] = g[i];
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < 32 * kQs; i += 64 * kWaves)
      lds.rows[i] = dev::toeplitz_word(lds.g, kWords, (int)(i / 32) + kQ0, dev::row_word(i % 32));
    __syncthreads();
  }

  // The jump of the pair whose states are s0 (in the pair's lanes, on every
  // wavefront), after lay_out: wavefront 0 runs the continuation, then each
  // wavefront multiplies a run of one stream's blocks and the shares are
  // added as words.  Thread 64 h + w, h < 2, returns word w of stream h.
  // Every thread of the workgroup calls it.
  static __device__ __forceinline__ typename M::word jump(const FamState<M> &s0, Lds &lds, const Lanes &L,
                                                          uint32_t wave) {
    using word = typename M::word;
    const uint32_t lane = L.lane;
    __syncthreads();  // an earlier jump's reads of s and part are done
    if (wave == 0) {
      auto put = [&](uint32_t c, word v) {
        lds.s[L.h][0][kStep * c + L.j] = (uint32_t)v;
        if constexpr (kPlanes == 2) lds.s[L.h][1][kStep * c + L.j] = (uint32_t)((uint64_t)v >> 32);
      };
      Ring2<M> g;
      g.open(s0.prev, s0.cur);
      put(0, s0.prev);
      put(1, s0.cur);
      const bool word0 = L.j == 0;
#pragma unroll 4
      for (uint32_t c = 2; c < 2 * kBlocks; ++c) put(c, g.step(word0));
    }
    __syncthreads();
    const dev::TransposeLane tl = dev::transpose_lane(lane);
    constexpr uint32_t kEach = kBlocks / kRuns, kMore = kBlocks % kRuns;  // the last kMore runs take one block more
    static_assert(kMore == 1, "the last run takes the odd block");
    const uint32_t h = wave & 1u, run = wave >> 1, c0 = kEach * run;
    const uint32_t *rows = lds.rows + 32 * (2 * c0 - kQ0) + lane;  // tile t of block c: q = 2 c - t + h'
    const uint32_t *bits = &lds.s[h][0][64 * c0 + lane];
    dev::tile_t acc[kPlanes][2] = {};
    auto block = [&]() {
      const dev::frag_t a0 = dev::frag(dev::one_bits(rows[0])), a1 = dev::frag(dev::one_bits(rows[-32]));
#pragma unroll
      for (uint32_t p = 0; p < kPlanes; ++p) {
        const dev::frag_t b = dev::frag(dev::half_bits(dev::word_bits(bits[64 * kBlocks * p], tl)));
        acc[p][0] = dev::mm_step(a0, b, acc[p][0]);
        acc[p][1] = dev::mm_step(a1, b, acc[p][1]);
      }
      rows += 64;
      bits += 64;
    };
#pragma unroll 4
    for (uint32_t i = 0; i < kEach; ++i) block();
    if (run == kRuns - 1) block();
#pragma unroll
    for (uint32_t p = 0; p < kPlanes; ++p) lds.part[wave][p][lane] = dev::tile_words(acc[p][0], acc[p][1], tl);
    __syncthreads();
    uint32_t y[2] = {0, 0};
    if (wave < 2) {
#pragma unroll
      for (uint32_t r = 0; r < kRuns; ++r)
#pragma unroll
        for (uint32_t p = 0; p < kPlanes; ++p) y[p] ^= lds.part[2 * r + wave][p][lane];
    }
    if constexpr (kPlanes == 2) return (uint64_t)y[0] | ((uint64_t)y[1] << 32);
    else return y[0];
  }
};

// Jumps by J: workgroups of 8 wavefronts, each taking every gridDim-th pair.
template <class M>
__global__ __launch_bounds__(FamJump<M>::kWaves * 64) void k_fam_skip_wg(unsigned char *__restrict__ state,
                                                                         uint64_t first, uint64_t count, uint64_t J,
                                                                         JumpPoly g) {
  using word = typename M::word;
  __shared__ typename FamJump<M>::Lds lds;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  FamJump<M>::lay_out(reinterpret_cast<const uint32_t *>(g.w), lds);
  for (uint64_t pair = blockIdx.x; 2 * pair < count; pair += gridDim.x) {
    const Lanes L = pair_lanes(pair, count);
    const FamState<M> s0 = fam_load<M>(state + (first + L.k) * M::state_bytes, true, L);
    const word y = FamJump<M>::jump(s0, lds, L, wave);
    if (wave < 2 && 2 * pair + wave < count) {
      unsigned char *st = state + (first + 2 * pair + wave) * M::state_bytes;
      reinterpret_cast<word *>(st)[L.lane] = y;
    }
    if (wave == 0 && L.j == 0) {
      unsigned char *st = state + (first + L.k) * M::state_bytes;
      *reinterpret_cast<word *>(st + M::weyl_off) = s0.weyl + (word)J * M::omega;
      *reinterpret_cast<uint64_t *>(st + M::pos_off) = s0.pos + J;
    }
  }
}

// Where part k of the launch's i-th stream keeps its start state: word t at
// out[i row + k part + (t / 32) chunk + t % 32]; W and pos follow the ring.
struct FamPlaces {
  uint64_t row, part, chunk;
};

template <class M>
__global__ __launch_bounds__(FamJump<M>::kWaves * 64) void k_fam_split_starts(
    const unsigned char *__restrict__ state, uint64_t first, uint32_t count, uint32_t exp,
    const uint64_t *__restrict__ table, typename M::word *__restrict__ out, FamPlaces at) {
  using word = typename M::word;
  __shared__ typename FamJump<M>::Lds lds;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t pairs = (count + 1) / 2, k = blockIdx.x / pairs, pair = blockIdx.x % pairs;
  const Lanes L = pair_lanes(pair, count);
  FamState<M> s0 = fam_load<M>(state + (first + L.k) * M::state_bytes, true, L);
  word *mine = out + L.k * at.row + k * at.part;
  if (k) {
    FamJump<M>::lay_out(reinterpret_cast<const uint32_t *>(table + (uint64_t)split_entry(exp, k) * (FamJump<M>::kWords / 2)),
                        lds);
    const word y = FamJump<M>::jump(s0, lds, L, wave);
    if (wave < 2 && 2 * pair + wave < count)
      out[(2 * pair + wave) * at.row + k * at.part + (L.lane / 32) * at.chunk + L.lane % 32] = y;
    const uint64_t by = (uint64_t)k << exp;
    s0.weyl += (word)by * M::omega;
    s0.pos += by;
  } else if (wave == 0) {
    mine[L.j] = s0.prev;
    mine[at.chunk + L.j] = s0.cur;
  }
  if (wave == 0 && L.j == 0) {
    word *w = mine + 2 * at.chunk;
    w[0] = s0.weyl;
    w[1] = (word)s0.pos;
    if constexpr (sizeof(word) == 4) w[2] = (word)(s0.pos >> 32);
  }
}

// One wavefront per part and pair of streams, from the states that
// k_fam_split_starts left; the last part writes the streams' end states.
template <class M, uint32_t KIND, bool FILL>
__global__ __launch_bounds__(256) void k_fam_split(unsigned char *__restrict__ state, uint64_t first, uint32_t count,
                                                   uint64_t n, uint32_t parts, uint32_t exp, typename M::word *out,
                                                   FamPlaces at) {
  using word = typename M::word;
  const uint32_t wid = (uint32_t)__builtin_amdgcn_readfirstlane((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
  const uint32_t pairs = (count + 1) / 2, k = wid / pairs, pair = wid % pairs;
  if (k >= parts) return;
  const Lanes L = pair_lanes(pair, count);
  const bool last = k + 1 == parts;
  const uint64_t done = (uint64_t)k << exp, nk = last ? n - done : 1ull << exp;
  word *o = out + L.k * at.row + k * at.part;
  const word *w = o + 2 * at.chunk;
  FamState<M> s0;
  s0.prev = o[L.j];
  s0.cur = o[at.chunk + L.j];
  s0.weyl = w[0];
  s0.pos = (uint64_t)w[1];
  if constexpr (sizeof(word) == 4) s0.pos |= (uint64_t)w[2] << 32;
  // Every word of the state is read before this wavefront writes over it.
  unsigned char *st = state + (first + L.k) * M::state_bytes;
  if constexpr (KIND == kNormal) {
    fam_normals_run<M, false, true, false>(s0, st, true, last, L, nk, reinterpret_cast<real_of<M> *>(o), nullptr);
  } else {
    word *tail = FILL ? out + (n / kStep) * at.chunk + L.k * (n % kStep) + L.j : nullptr;
    fam_run<M, KIND, 8, false>(s0, st, true, last, L, nk, o + L.j, FILL ? at.chunk : kStep, tail);
  }
}

template <class M>
hipError_t launch_fam_split(Kind kind, bool fill, const Split &sp, unsigned char *state, uint64_t first,
                            uint64_t count, uint64_t n, const uint64_t *table, void *out, int num_cus,
                            hipStream_t stream) {
  using word = typename M::word;
  constexpr uint32_t kInt = sizeof(word) == 4 ? kU32 : kU64, kReal = sizeof(word) == 4 ? kF32 : kF64;
  const uint64_t waves = (count + 1) / 2 * sp.parts;
  const uint64_t wpb = auto_waves_per_block(waves, num_cus);
  word *o = static_cast<word *>(out);
  const uint64_t part = 1ull << sp.exp;
  const FamPlaces at = fill ? FamPlaces{kStep, part * count, kStep * count} : FamPlaces{n, part, kStep};
  hipError_t e = launch(k_fam_split_starts<M>, dim3((uint32_t)waves), dim3(FamJump<M>::kWaves * 64), 0, stream, state,
                        first, count, sp.exp, table, o, at);
  if (e != hipSuccess) return e;
  auto run = [&](auto kernel) {
    return launch(kernel, dim3((uint32_t)((waves + wpb - 1) / wpb)), dim3((uint32_t)(wpb * kWave)), 0, stream, state,
                  first, count, n, sp.parts, sp.exp, o, at);
  };
  if (kind == kNormal) return run(k_fam_split<M, kNormal, false>);
  if (kind == kReal) return fill ? run(k_fam_split<M, kReal, true>) : run(k_fam_split<M, kReal, false>);
  if (kind == kInt) return fill ? run(k_fam_split<M, kInt, true>) : run(k_fam_split<M, kInt, false>);
  return hipErrorInvalidValue;
}

template <class M, uint32_t KIND, bool FILL, bool NT>
hipError_t launch_fam_k(uint32_t unroll, dim3 grid, dim3 block, unsigned char *state, uint64_t first,
                  uint64_t count, uint64_t n, void *out, hipStream_t stream) {
  auto run = [&](auto kernel) { return launch(kernel, grid, block, 0, stream, state, first, count, n, out); };
  switch (unroll) {
    case 1: return run(k_fam_generate<M, KIND, 1, FILL, NT>);
    case 2: return run(k_fam_generate<M, KIND, 2, FILL, NT>);
    case 4: return run(k_fam_generate<M, KIND, 4, FILL, NT>);
    default: return run(k_fam_generate<M, KIND, 8, FILL, NT>);
  }
}

// The bulk-fill layout takes non-temporal stores, stream-major rows those of cached_stores.
template <class M, uint32_t KIND>
hipError_t launch_fam_layout(bool fill, bool cached, uint32_t unroll, dim3 grid, dim3 block, unsigned char *state,
                             uint64_t first, uint64_t count, uint64_t n, void *out, hipStream_t stream) {
  if (fill) return launch_fam_k<M, KIND, true, true>(unroll, grid, block, state, first, count, n, out, stream);
  if (cached) return launch_fam_k<M, KIND, false, false>(unroll, grid, block, state, first, count, n, out, stream);
  return launch_fam_k<M, KIND, false, true>(unroll, grid, block, state, first, count, n, out, stream);
}

// The 32-bit member's normals with more than a wavefront per SIMD gather their
// pairs through LDS, which takes selects and swaps off the VALU (3001 streams x
// 65537: 235 us and 204; moments of 4096 x 2^16: 233 and 218).  One wavefront
// per SIMD waits for the LDS instead (2048 x 2^17: normals 278 us and 290,
// moments 247 and 300), and the 64-bit member gains nothing from it (4096 x
// 2^16: normals 552 and 556).
template <class M>
hipError_t launch_fam_normals(Kind kind, bool nt, uint64_t pairs, int num_cus, dim3 grid, dim3 block,
                              unsigned char *state, uint64_t first, uint64_t count, uint64_t n, void *out,
                              hipStream_t stream) {
  auto run = [&](auto kernel, size_t lds) {
    return launch(kernel, grid, block, lds, stream, state, first, count, n, kind == kNormal ? out : nullptr,
                  kind == kMoments ? out : nullptr);
  };
  if constexpr (sizeof(typename M::word) == 4) {
    if (pairs > 4 * (uint64_t)(num_cus > 0 ? num_cus : 1)) {
      const size_t lds = (size_t)block.x / kWave * 2 * kFamStage * sizeof(typename M::word);
      return kind == kMoments ? run(k_fam_normals<M, true, false, true>, lds)
             : nt             ? run(k_fam_normals<M, false, true, true>, lds)
                              : run(k_fam_normals<M, false, false, true>, lds);
    }
  }
  return kind == kMoments ? run(k_fam_normals<M, true, false, false>, 0)
         : nt             ? run(k_fam_normals<M, false, true, false>, 0)
                          : run(k_fam_normals<M, false, false, false>, 0);
}

}  // namespace

uint32_t family_state_bytes(uint32_t family) {
  switch (family) {
    case XG_FAMILY_R128_W32: return XG_STATE_WORDS * 4;
    case XG_FAMILY_R64_W32: return MemberN2048::state_bytes;
    case XG_FAMILY_R64_W64: return MemberW64::state_bytes;
    default: return 0;
  }
}

uint32_t family_pos_offset(uint32_t family) {
  switch (family) {
    case XG_FAMILY_R128_W32: return 130 * 4;
    case XG_FAMILY_R64_W32: return MemberN2048::pos_off;
    case XG_FAMILY_R64_W64: return MemberW64::pos_off;
    default: return 0;
  }
}

hipError_t launch_family_init(uint32_t family, unsigned char *state, uint64_t num_streams, uint64_t seed,
                              hipStream_t stream) {
  hipError_t e = hipSuccess;
  const uint64_t pairs = (num_streams + 1) / 2;
  const dim3 grid((uint32_t)((pairs + 3) / 4)), block(256);
  if (family == XG_FAMILY_R64_W32)
    e = launch(k_fam_init<MemberN2048>, grid, block, 0, stream, state, num_streams, seed);
  else if (family == XG_FAMILY_R64_W64)
    e = launch(k_fam_init<MemberW64>, grid, block, 0, stream, state, num_streams, seed);
  else
    return hipErrorInvalidValue;
  return e;
}

hipError_t launch_family_skip(uint32_t family, unsigned char *state, uint64_t first, uint64_t count, uint64_t J,
                              const JumpPoly *g, int num_cus, hipStream_t stream) {
  hipError_t e = hipSuccess;
  const uint64_t pairs = (count + 1) / 2, cus = num_cus > 0 ? (uint64_t)num_cus : 1;
  const dim3 grid((uint32_t)((pairs + 3) / 4)), block(256);
  JumpPoly zero{};
  const JumpPoly &gp = g ? *g : zero;
  // The matrix-core form while a workgroup takes at most a few pairs of
  // streams: its continuation runs on one wavefront, where the other form runs
  // one per pair (us, this form and the other: 32-bit member 1024 streams 9,
  // 25; 4096 28, 29; 8192 52, 49; 64-bit member 1024 28, 78; 2048 51, 79; 4096
  // 96, 91).
  if (g && pairs <= (family == XG_FAMILY_R64_W32 ? 8 : 6) * cus) {
    const dim3 wgrid((uint32_t)(pairs < 2 * cus ? pairs : 2 * cus));
    auto run = [&](auto kernel, uint32_t waves) {
      return launch(kernel, wgrid, dim3(waves * 64), 0, stream, state, first, count, J, gp);
    };
    if (family == XG_FAMILY_R64_W32) return run(k_fam_skip_wg<MemberN2048>, FamJump<MemberN2048>::kWaves);
    if (family == XG_FAMILY_R64_W64) return run(k_fam_skip_wg<MemberW64>, FamJump<MemberW64>::kWaves);
    return hipErrorInvalidValue;
  }
  if (family == XG_FAMILY_R64_W32) {
    if (g) e = launch((k_fam_skip<MemberN2048, true>), grid, block, 4 * 192 * 4, stream, state, first, count, J, gp);
    else e = launch((k_fam_skip<MemberN2048, false>), grid, block, 0, stream, state, first, count, J, gp);
  } else if (family == XG_FAMILY_R64_W64) {
    if (g) e = launch((k_fam_skip<MemberW64, true>), grid, block, 4 * 192 * 8, stream, state, first, count, J, gp);
    else e = launch((k_fam_skip<MemberW64, false>), grid, block, 0, stream, state, first, count, J, gp);
  } else {
    return hipErrorInvalidValue;
  }
  return e;
}

hipError_t launch_family_split(uint32_t family, Kind kind, bool fill, const Split &sp, unsigned char *state,
                               uint64_t first, uint64_t count, uint64_t n, const uint64_t *table, void *out,
                               int num_cus, hipStream_t stream) {
  if (family == XG_FAMILY_R64_W32)
    return launch_fam_split<MemberN2048>(kind, fill, sp, state, first, count, n, table, out, num_cus, stream);
  if (family == XG_FAMILY_R64_W64)
    return launch_fam_split<MemberW64>(kind, fill, sp, state, first, count, n, table, out, num_cus, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_family_generate(uint32_t family, Kind kind, bool fill, const Shape &shape, unsigned char *state,
                                  uint64_t first, uint64_t count, uint64_t n, void *out, int num_cus,
                                  hipStream_t stream) {
  hipError_t e = hipSuccess;
  const uint64_t pairs = (count + 1) / 2;
  const uint64_t wpb = shape.waves_per_block;
  const dim3 grid((uint32_t)((pairs + wpb - 1) / wpb)), block((uint32_t)(wpb * kWave));
  const bool cached = cached_stores(family, kind, count, n, reinterpret_cast<uintptr_t>(out), num_cus);
  if (kind == kNormal || kind == kMoments) {
    const bool nt = kind == kNormal && !cached;
    if (family == XG_FAMILY_R64_W32)
      return launch_fam_normals<MemberN2048>(kind, nt, pairs, num_cus, grid, block, state, first, count, n, out, stream);
    if (family == XG_FAMILY_R64_W64)
      return launch_fam_normals<MemberW64>(kind, nt, pairs, num_cus, grid, block, state, first, count, n, out, stream);
    return hipErrorInvalidValue;
  }
  if (family == XG_FAMILY_R64_W32 && kind == kU32)
    e = launch_fam_layout<MemberN2048, kU32>(fill, cached, shape.unroll, grid, block, state, first, count, n, out, stream);
  else if (family == XG_FAMILY_R64_W32 && kind == kF32)
    e = launch_fam_layout<MemberN2048, kF32>(fill, cached, shape.unroll, grid, block, state, first, count, n, out, stream);
  else if (family == XG_FAMILY_R64_W64 && kind == kU64)
    e = launch_fam_layout<MemberW64, kU64>(fill, cached, shape.unroll, grid, block, state, first, count, n, out, stream);
  else if (family == XG_FAMILY_R64_W64 && kind == kF64)
    e = launch_fam_layout<MemberW64, kF64>(fill, cached, shape.unroll, grid, block, state, first, count, n, out, stream);
  else
    return hipErrorInvalidValue;
  return e;
}

// Groups per compute unit up to which there is a wavefront for each (see
// look_at_pairs; 1500 requests of mixed types and 2^8 to 2^14 words: 81 us in pairs
// and 64, 2000 81 and 72, and more than two wavefronts per SIMD gain nothing).
constexpr uint64_t kAlone = 8;
hipError_t launch_family_batch(uint32_t family, const Shape &shape, int num_cus, unsigned char *state,
                               uint64_t num_streams, const xg_request *reqs, const uint32_t *groups,
                               uint32_t max_groups, void *out, uint64_t out_elems, uint32_t *work,
                               hipStream_t stream) {
  if (family != XG_FAMILY_R64_W32 && family != XG_FAMILY_R64_W64) return hipErrorInvalidValue;
  hipError_t e = hipSuccess;
  const uint64_t cus = num_cus > 0 ? num_cus : 1;
  const uint64_t items = max_groups <= kAlone * cus ? max_groups : ((uint64_t)max_groups + 1) / 2;
  uint64_t blocks = cus * shape.blocks_per_cu;
  const uint64_t need = (items + shape.waves_per_block - 1) / shape.waves_per_block;
  if (need < blocks) blocks = need ? need : 1;
  const dim3 block(shape.waves_per_block * kWave);
  if (family == XG_FAMILY_R64_W32)
    e = launch_fam_batch_k<MemberN2048>(shape.unroll, blocks, block, num_cus, state, num_streams, reqs, groups, out,
                                        out_elems, work, stream);
  else
    e = launch_fam_batch_k<MemberW64>(shape.unroll, blocks, block, num_cus, state, num_streams, reqs, groups, out,
                                      out_elems, work, stream);
  return e;
}

}  // namespace xg
