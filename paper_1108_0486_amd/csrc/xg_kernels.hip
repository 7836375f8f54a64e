// HIP kernels of libxg for gfx950 (MI355X): xorgens streams, one wavefront per
// stream, 64 consecutive words per wavefront step.
//
// Method (arXiv:1108.0486):
//   Section 2       x_i = x_{i-128} A  xor  x_{i-65} B,
//                   A = (I + L^15)(I + R^14), B = (I + L^12)(I + R^17), 32-bit words;
//   Section 1.5     W_k = W_{k-1} + omega,  out_k = x_k + (W_k xor (W_k >> 16))  (Eq. (1));
//   Section 2       x_k .. x_{k+C-1} depend only on words older than x_k while
//                   C <= s = 65, so one 64-lane wavefront computes 64 words per step.
//
// Register-resident ring.  Lane j of a wavefront owns word j of every 64-word
// chunk.  For the chunk starting at position p the wavefront holds
//   prev[j] = x_{p-128+j}   (chunk p-128 .. p-65)
//   cur[j]  = x_{p-64+j}    (chunk p-64  .. p-1)
// and computes x_{p+j} = A(prev[j]) xor B(x_{p+j-65}).  Here x_{p+j-65} is
// cur[j-1] for j >= 1 and prev[63] for j = 0: B(cur) is rotated up by one lane
// with a DPP wave rotate, and lane 0 takes B(prev[63]), which is lane 0 of the
// previous chunk's rotation.  The 128-word ring thus never leaves VGPRs inside
// the hot loop; each chunk costs about 14 VALU operations per lane and one
// coalesced 256-byte store.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xg_device.h"
#include "xg_jump_mm.h"
#include "xg_normal.h"
#include "xg_internal.h"
#include "xg_launch.h"

namespace xg {
namespace {

using dev::box_muller;
using dev::box_muller_unordered;
using dev::group_add;
using dev::group_close;
using dev::lanes_rotate_up;
using dev::Moments;
using dev::wave_lds_sync;
using dev::splitmix64_at;
using dev::xcd_block;
using dev::xor3;

constexpr uint32_t kOmega = 0x9E3779B9u;       // odd integer nearest 2^31 (sqrt 5 - 1)
constexpr uint32_t kChunkOmega = 64u * kOmega;  // Weyl advance per chunk (mod 2^32)

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));

// x (I + L^12)(I + R^17): the operator applied to x_{i-s}.
__device__ __forceinline__ uint32_t op_lag_s(uint32_t v) {
  v ^= v << 12;
  return v ^ (v >> 17);
}

__device__ __forceinline__ uint32_t temper_weyl(uint32_t w) { return w ^ (w >> 16); }

struct Ring {
  uint32_t prev;   // x_{p-128+j}
  uint32_t cur;    // x_{p-64+j}
  uint32_t rprev;  // lane 0: B(x_{p-65}); other lanes: unused
};

__device__ __forceinline__ Ring ring_from(uint32_t prev, uint32_t cur) {
  Ring g;
  g.prev = prev;
  g.cur = cur;
  g.rprev = lanes_rotate_up(op_lag_s(prev));  // lane 0 <- B(prev[63]) = B(x_{p-65})
  return g;
}

// Computes the next 64 words x_p .. x_{p+63} (lane j: x_{p+j}) and advances g.
__device__ __forceinline__ uint32_t ring_step(Ring &g, bool lane0) {
  const uint32_t bc = op_lag_s(g.cur);
  const uint32_t rc = lanes_rotate_up(bc);     // lane j >= 1: B(x_{p+j-65}); lane 0: B(x_{p-1})
  const uint32_t bs = lane0 ? g.rprev : rc;    // B(x_{p+j-65}) on every lane
  // A(prev) = prev (I + L^15)(I + R^14) = t xor (t >> 14), t = prev xor (prev << 15)
  const uint32_t t = g.prev ^ (g.prev << 15);
  const uint32_t x = xor3(t, t >> 14, bs);
  g.prev = g.cur;
  g.cur = x;
  g.rprev = rc;                                // lane 0: B(x_{p-1}) = B(x_{p'-65}), p' = p + 64
  return x;
}

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & (kWave - 1); }


// Makes prev | cur the 128-word window ending `rem` words into chunk `x` (rem
// in 1..63), i.e. words [rem, rem + 128) of the concatenation prev | cur | x;
// rem == 0 leaves them.
__device__ __forceinline__ void turn_ring(uint32_t &prev, uint32_t &cur, uint32_t x, uint32_t rem, uint32_t lane) {
  if (rem) {
    const int src = (int)((rem + lane) & 63u);
    const uint32_t a = (uint32_t)__shfl((int)prev, src);
    const uint32_t b = (uint32_t)__shfl((int)cur, src);
    const uint32_t c = (uint32_t)__shfl((int)x, src);
    const bool wrap = rem + lane >= 64u;
    prev = wrap ? b : a;
    cur = wrap ? c : b;
  }
}

// Writes that window as the new linear ring.
__device__ __forceinline__ void store_ring(uint32_t *st, uint32_t prev, uint32_t cur, uint32_t x,
                                           uint32_t rem, uint32_t lane) {
  turn_ring(prev, cur, x, rem, lane);
  st[lane] = prev;
  st[64 + lane] = cur;
}

__device__ __forceinline__ void store_weyl_pos(uint32_t *st, uint32_t weyl, uint64_t pos,
                                               uint32_t lane) {
  if (lane == 0) {
    st[128] = weyl;
    st[129] = 0u;
    st[130] = (uint32_t)pos;
    st[131] = (uint32_t)(pos >> 32);
  }
}

__device__ __forceinline__ uint64_t load_pos(const uint32_t *st) {
  return (uint64_t)st[130] | ((uint64_t)st[131] << 32);
}

// Output word of type KIND for generator output o (FP32 as its bit pattern):
// u32 as is; f32 (o >> 8) * 2^-24, exact (a 24-bit integer times a power of two).
template <uint32_t KIND>
__device__ __forceinline__ uint32_t map_word(uint32_t o) {
  if constexpr (KIND == kU32) {
    return o;
  } else {
    return __float_as_uint((float)(o >> 8) * 0x1p-24f);
  }
}

// PACED: the store is followed by an issue gap of three wait states
// (s_nop 2).  Used only by the uint32 stream-major launch at unroll 2 with
// 4-byte stores: there, with one wavefront per SIMD and 1024 fronts 4 MB
// apart, spacing each wavefront's 256-byte stores this way took a 4 GiB
// launch from 790-815 us to 717-736 us on three boxes (interleaved A/B), as
// fast as the FP32 launch, whose three extra ALU operations per chunk space
// its stores anyway.  Longer gaps, other unrolls and the other layouts
// measured slower with it, so nothing else is paced.
//
// NT: a non-temporal store (the plain launches, whose rows start aligned);
// otherwise a plain one (the batch kernel: with dense output offsets most
// requests start inside a cache line, and plain stores let the L2 merge the
// partial lines at both ends of every wavefront's 256-byte store, where
// non-temporal ones took the ragged batch from 7.1 to 12.7 ms).
//
// Loops that unroll by UNROLL write UNROLL = 1 without the one-trip inner
// loop: LLVM's LICM promotes the store of a one-trip inner loop to the loop's
// exit, and the promoted store no longer carries the non-temporal hint.
template <bool NT, class T>
__device__ __forceinline__ void store_out(T v, T *p) {
  if constexpr (NT) {
    __builtin_nontemporal_store(v, p);
  } else {
    *p = v;
  }
}

template <uint32_t KIND, bool PACED = false, bool NT = true>
__device__ __forceinline__ void emit_word(uint32_t *p, uint32_t o) {
  store_out<NT>(map_word<KIND>(o), p);
  if constexpr (PACED) asm volatile("s_nop 2");
}

// Dynamic LDS: one 256-word staging slot per wavefront of the block (wide stores).
extern __shared__ __align__(16) uint32_t xg_lds[];

__device__ __forceinline__ uint32_t *wave_stage() { return xg_lds + (threadIdx.x >> 6) * 256u; }
// The normals' two slots per wavefront.
__device__ __forceinline__ uint32_t *normals_stage() { return xg_lds + (threadIdx.x >> 6) * 512u; }


// ---------------------------------------------------------------------------
// A stream's state held by a wavefront: lane j has ring words j and 64 + j;
// the Weyl value W_{pos-1} and the position are wave-uniform.
// ---------------------------------------------------------------------------
struct StreamState {
  uint32_t prev;  // x_{pos-128+j}
  uint32_t cur;   // x_{pos-64+j}
  uint32_t weyl;  // W_{pos-1}
  uint64_t pos;
};

__device__ __forceinline__ StreamState load_state(const uint32_t *st) {
  const uint32_t lane = lane_id();
  StreamState s;
  s.prev = st[lane];
  s.cur = st[64 + lane];
  s.weyl = st[128];
  s.pos = load_pos(st);
  return s;
}

// Writes the state whose ring is the 128-word window ending `rem` words into
// chunk x (see store_ring); dst == nullptr (wave-uniform) writes nothing.
__device__ __forceinline__ void write_state(uint32_t *dst, uint32_t prev, uint32_t cur, uint32_t x,
                                            uint32_t rem, uint32_t weyl, uint64_t pos, uint32_t lane) {
  if (!dst) return;
  store_ring(dst, prev, cur, x, rem, lane);
  store_weyl_pos(dst, weyl, pos, lane);
}

// Where a request's end state goes, a window as in write_state: to memory (or
// nowhere), or into registers for the stream's next request.
struct ToMemory {
  uint32_t *dst;
  __device__ __forceinline__ void operator()(uint32_t prev, uint32_t cur, uint32_t x, uint32_t rem, uint32_t weyl,
                                             uint64_t pos, uint32_t lane) const {
    write_state(dst, prev, cur, x, rem, weyl, pos, lane);
  }
};
struct ToRegisters {
  StreamState *s;
  __device__ __forceinline__ void operator()(uint32_t prev, uint32_t cur, uint32_t x, uint32_t rem, uint32_t weyl,
                                             uint64_t pos, uint32_t lane) const {
    turn_ring(prev, cur, x, rem, lane);
    *s = StreamState{prev, cur, weyl, pos};
  }
};

// ---------------------------------------------------------------------------
// One stream's word sequence inside a wavefront: open (from a state), next
// (one 64-word chunk of outputs, lane j holding word j), close (the ragged last
// chunk, then the state write-back).
// ---------------------------------------------------------------------------
struct WordStream {
  Ring g;
  uint32_t w_start;  // W_{pos-1} at open
  uint32_t wbase;    // W_{p-1} for the next chunk at p
  uint32_t wlane;    // (j + 1) omega: W_{p+j} = W_{p-1} + (j + 1) omega
  uint64_t pos;
  uint32_t lane;
  bool lane0;
};

__device__ __forceinline__ WordStream open_from(const StreamState &st) {
  WordStream s;
  s.lane = lane_id();
  s.lane0 = s.lane == 0;
  s.g = ring_from(st.prev, st.cur);
  s.w_start = st.weyl;
  s.wbase = s.w_start;
  s.wlane = (s.lane + 1u) * kOmega;
  s.pos = st.pos;
  return s;
}

__device__ __forceinline__ WordStream open_stream(const uint32_t *st) { return open_from(load_state(st)); }

__device__ __forceinline__ uint32_t next_chunk(WordStream &s) {
  const uint32_t x = ring_step(s.g, s.lane0);
  const uint32_t w = s.wbase + s.wlane;
  s.wbase += kChunkOmega;
  return x + temper_weyl(w);
}

// Emits the last rem (< 64) words of an n-word request through `tail`
// (lane-indexed: lane j writes tail[j], j < rem) and hands the end state to `end`.
template <uint32_t KIND, bool NT = true, class End>
__device__ __forceinline__ void close_stream(End end, WordStream &s, uint64_t n, uint32_t rem,
                                             uint32_t *tail) {
  const uint32_t p0 = s.g.prev, c0 = s.g.cur;
  uint32_t x = 0u;
  if (rem) {
    x = ring_step(s.g, s.lane0);
    const uint32_t w = s.wbase + s.wlane;
    if (s.lane < rem) emit_word<KIND, false, NT>(tail, x + temper_weyl(w));
  }
  end(p0, c0, x, rem, s.w_start + (uint32_t)n * kOmega, s.pos + n, s.lane);
}

// ---------------------------------------------------------------------------
// u32 / f32, stream-major: n words of one stream written at out[0 .. n).
// WIDE: while out is 16-byte aligned, four chunks (256 words) are staged in
// the wavefront's LDS slot and leave as one 16-byte store per lane (1 KB per
// store instruction instead of 256 B); the rest uses one 4-byte store per lane.
// ---------------------------------------------------------------------------
template <uint32_t KIND, int UNROLL, bool WIDE, bool PACED = false, bool NT = true, class End>
__device__ __forceinline__ void serve_words_from(const StreamState &s0, uint64_t n, uint32_t *__restrict__ out,
                                                 End end) {
  WordStream s = open_from(s0);
  const uint32_t lane = s.lane;
  const uint64_t nfull = n >> 6;
  const uint32_t rem = (uint32_t)(n & 63u);
  uint64_t done = 0;  // chunks written by the wide loop
  if constexpr (WIDE) {
    static_assert(UNROLL % 4 == 0, "wide stores take groups of four chunks");
    if ((reinterpret_cast<uintptr_t>(out) & 15u) == 0) {
      uint32_t *stage = wave_stage();
      u32x4 *o4 = reinterpret_cast<u32x4 *>(out) + lane;
      const uint64_t nouter = nfull / UNROLL;
      for (uint64_t it = 0; it != nouter; ++it) {
#pragma unroll
        for (int q = 0; q < UNROLL / 4; ++q) {
#pragma unroll
          for (int u = 0; u < 4; ++u) stage[64 * u + lane] = map_word<KIND>(next_chunk(s));
          wave_lds_sync();  // the read below takes words other lanes wrote
          const u32x4 v = *reinterpret_cast<const u32x4 *>(stage + 4 * lane);
          wave_lds_sync();  // the next group's writes come after this read
          store_out<NT>(v, o4 + q * 64);
        }
        o4 += (UNROLL / 4) * 64;
      }
      done = nouter * UNROLL;
    }
  }
  uint32_t *o = out + done * 64 + lane;
  const uint64_t nrest = nfull - done;
  const uint64_t nouter = nrest / UNROLL;
  for (uint64_t it = 0; it != nouter; ++it) {
    if constexpr (UNROLL == 1) {
      emit_word<KIND, PACED, NT>(o, next_chunk(s));
    } else {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) emit_word<KIND, PACED, NT>(o + u * 64, next_chunk(s));
    }
    o += UNROLL * 64;
  }
  const uint32_t nleft = (uint32_t)(nrest % UNROLL);
  for (uint32_t c = 0; c != nleft; ++c) {
    emit_word<KIND, PACED, NT>(o, next_chunk(s));
    o += 64;
  }
  close_stream<KIND, NT>(end, s, n, rem, o);
}

template <uint32_t KIND, int UNROLL, bool WIDE, bool PACED = false>
__device__ __forceinline__ void serve_words(uint32_t *st, uint64_t n, uint32_t *__restrict__ out) {
  serve_words_from<KIND, UNROLL, WIDE, PACED>(load_state(st), n, out, ToMemory{st});
}

// ---------------------------------------------------------------------------
// u32 / f32, bulk-fill layout: chunk c (words 64c .. 64c + 63) of the k-th of
// `count` streams goes to out[(c count + k) 64 ..], so the wavefronts of a
// launch write one dense, advancing region of HBM instead of `count` fronts
// n words apart; the ragged last chunks (rem = n mod 64 words each) follow,
// packed, at out[64 (n / 64) count + k rem ..].  The values are those of the
// stream-major layout; only their places differ.
// ---------------------------------------------------------------------------
template <uint32_t KIND, int UNROLL, bool NT = true>
__device__ __forceinline__ void serve_chunks(const StreamState &s0, uint64_t n, uint32_t *o, uint64_t stride,
                                             uint32_t *tail, uint32_t *dst) {
  WordStream s = open_from(s0);
  const uint64_t nfull = n >> 6;
  const uint32_t rem = (uint32_t)(n & 63u);
  const uint64_t nouter = nfull / UNROLL;
  for (uint64_t it = 0; it != nouter; ++it) {
    if constexpr (UNROLL == 1) {
      emit_word<KIND, false, NT>(o, next_chunk(s));
    } else {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) emit_word<KIND, false, NT>(o + u * stride, next_chunk(s));
    }
    o += UNROLL * stride;
  }
  const uint32_t nleft = (uint32_t)(nfull % UNROLL);
  for (uint32_t c = 0; c != nleft; ++c) {
    emit_word<KIND, false, NT>(o, next_chunk(s));
    o += stride;
  }
  close_stream<KIND, NT>(ToMemory{dst}, s, n, rem, tail);
}

template <uint32_t KIND, int UNROLL>
__device__ __forceinline__ void serve_words_fill(uint32_t *__restrict__ st, uint64_t n, uint64_t k,
                                                 uint64_t count, uint32_t *__restrict__ out) {
  const uint32_t lane = lane_id();
  const uint64_t nfull = n >> 6;
  const uint32_t rem = (uint32_t)(n & 63u);
  const uint64_t stride = count * 64;
  serve_chunks<KIND, UNROLL>(load_state(st), n, out + k * 64 + lane, stride,
                             out + nfull * stride + k * rem + lane, st);
}

// ---------------------------------------------------------------------------
// normals: Box-Muller on consecutive output pairs of the call.
// ---------------------------------------------------------------------------
// Two ways to give the lanes their pairs of consecutive words.
//  - LDS: two 128-word blocks are written to the wavefront's LDS a chunk at a
//    time and read back four consecutive words per lane, two pairs, whose
//    normals leave as one 16-byte store (consume_quad).  No VALU instruction,
//    for launches with more than one wavefront per SIMD, where the VALU is the
//    bound and the LDS latency hides: 4096 x 2^18 normals 825 us and moments
//    722 (870 and 738 with one block at a time by four ds_bpermute and two
//    selects, which gather_pair does for what the unrolled loop leaves over; on
//    a slower box normals 863 and 906).
//  - DPP (an even lane j takes words j and j + 1, an odd lane j words 63 + j
//    and 64 + j): each lane needs one word of its neighbour in the same chunk,
//    which a quad permutation (lanes 2i and 2i + 1 swap) supplies in the VALU,
//    with no LDS round trip to wait for.
// DPP and LDS in us at 2^19 per stream: 1024 streams normals 489 and 507, moments
// 462 and 502; 1536 streams 811 and 745, 890 and 776; 2048 streams 890 and 851,
// 894 and 779.  So the line is one wavefront per SIMD.
// pair_offset gives the first word of a gather_pair pair within the block.
template <bool DPP>
__device__ __forceinline__ uint32_t pair_offset(uint32_t lane) {
  return DPP ? (lane & ~1u) + ((lane & 1u) << 6) : 2u * lane;
}

template <bool DPP>
__device__ __forceinline__ void gather_pair(uint32_t lo, uint32_t hi, uint32_t lane, uint32_t &e, uint32_t &o) {
  if constexpr (DPP) {
    // Bit selects, not ternaries, so that the swaps cannot be sunk into
    // lane-divergent branches where the neighbouring lanes are inactive.
    constexpr int kSwapPairs = 0xB1;  // quad_perm [1, 0, 3, 2]
    const uint32_t odd = 0u - (lane & 1u);  // all ones on odd lanes
    const uint32_t lo_sw = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo, kSwapPairs, 0xF, 0xF, false);
    const uint32_t hi_sw = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, kSwapPairs, 0xF, 0xF, false);
    e = dev::select_bits(hi_sw, lo, odd);
    o = dev::select_bits(hi, lo_sw, odd);
  } else {
    const int se = (int)((2u * lane) & 63u);
    const int so = se + 1;
    const uint32_t e_lo = (uint32_t)__shfl((int)lo, se), e_hi = (uint32_t)__shfl((int)hi, se);
    const uint32_t o_lo = (uint32_t)__shfl((int)lo, so), o_hi = (uint32_t)__shfl((int)hi, so);
    const bool upper = lane >= 32u;
    e = upper ? e_hi : e_lo;
    o = upper ? o_hi : o_lo;
  }
}

// Stores (or accumulates) normals idx and idx + 1 of the call.  CHECKED
// compares them with n (blocks wholly inside n skip that).  The two adjacent
// 4-byte stores of a full pair become one 8-byte store, which needs only
// 4-byte alignment.
template <bool MOMENTS, bool CHECKED, bool NT = true>
__device__ __forceinline__ void consume_pair(uint32_t e, uint32_t o, uint64_t idx, uint64_t n,
                                             float *__restrict__ out, Moments &m) {
  float z0, z1;
  if constexpr (MOMENTS && !CHECKED) {
    box_muller_unordered(e, o, z0, z1);  // a whole pair into the sums: its order is immaterial
  } else {
    box_muller(e, o, z0, z1);
  }
  const bool has0 = !CHECKED || idx < n, has1 = !CHECKED || idx + 1 < n;
  if constexpr (MOMENTS) {
    // Into the open group (the caller closes groups); has1 implies has0.
    if (has0) group_add(m, z0, has1 ? z1 : 0.0f);
  } else {
    if (has0) store_out<NT>(z0, out + idx);
    if (has1) store_out<NT>(z1, out + idx + 1);
  }
}

// The two pairs of four consecutive words: their four normals stored at out, or
// added to the open group.  The store needs the alignment of one value only.
template <bool MOMENTS, bool NT = true>
__device__ __forceinline__ void consume_quad(u32x4 w, float *out, Moments &m) {
  f32x4 z;
  if constexpr (MOMENTS) {
    float a, b;
    box_muller_unordered(w.x, w.y, a, b);
    group_add(m, a, b);
    box_muller_unordered(w.z, w.w, a, b);
    group_add(m, a, b);
  } else {
    float a, b;
    box_muller(w.x, w.y, a, b);
    z.x = a;
    z.y = b;
    box_muller(w.z, w.w, a, b);
    z.z = a;
    z.w = b;
    f32x4 *o = reinterpret_cast<f32x4 *>(out);
    if constexpr (NT) __builtin_nontemporal_store(z, o);
    else *o = z;
  }
}

// n normals of one stream; MOMENTS: reduce to (sum z, sum z^2) in sums[0..1]
// instead of storing them.  Consumes 2 ceil(n / 2) words.  DPP picks the
// pair gather (above).
template <bool MOMENTS, int UNROLL, bool DPP, bool NT = true, class End>
__device__ __forceinline__ void serve_normals_from(const StreamState &s0, uint64_t n, float *__restrict__ out,
                                                   float *__restrict__ sums, End end) {
  const uint32_t lane = lane_id();
  const bool lane0 = lane == 0;
  Ring g = ring_from(s0.prev, s0.cur);
  const uint32_t w_start = s0.weyl;
  const uint64_t pos = s0.pos;
  uint32_t wbase = w_start;
  const uint32_t wlane = (lane + 1u) * kOmega;
  const uint64_t words = n + (n & 1u);
  const uint64_t nblk = words >> 7;     // 128-word blocks: 64 pairs, one per lane
  const uint32_t rw = (uint32_t)(words & 127u);
  Moments m = {0.f, 0.f, 0.f, 0.f, -0.f, -0.f};
  const uint64_t nsafe = n >> 7;        // blocks whose 128 normals are all below n
  const uint32_t poff = pair_offset<DPP>(lane);
  const uint64_t nouter = UNROLL > 1 ? nsafe / UNROLL : 0;  // UNROLL = 1: the loop after this one
  uint64_t b = 0;
  auto next_word = [&]() {
    const uint32_t x = ring_step(g, lane0);
    const uint32_t w = x + temper_weyl(wbase + wlane);
    wbase += kChunkOmega;
    return w;
  };
  for (uint64_t it = 0; it != nouter; ++it, b += UNROLL) {
    if constexpr (!DPP && UNROLL > 1) {
#pragma unroll
      for (int u = 0; u < UNROLL; u += 2) {  // two blocks: four words, so two pairs, per lane
        uint32_t *stage = normals_stage() + 256u * ((u / 2) & 1);
#pragma unroll
        for (int c = 0; c < 4; ++c) stage[64 * c + lane] = next_word();
        wave_lds_sync();  // the read below takes words other lanes wrote
        const u32x4 w = *reinterpret_cast<const u32x4 *>(stage + 4 * lane);
        wave_lds_sync();  // the next writes to this half come after this read
        consume_quad<MOMENTS, NT>(w, out + (((b + u) << 7) + 4 * lane), m);
        if (MOMENTS && ((u & 2) || u == UNROLL - 2)) group_close(m);
      }
    } else {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        const uint32_t oa = next_word();
        const uint32_t ob = next_word();
        uint32_t e, o;
        gather_pair<DPP>(oa, ob, lane, e, o);
        consume_pair<MOMENTS, false, NT>(e, o, ((b + u) << 7) + poff, n, out, m);
        if (MOMENTS && ((u & 3) == 3 || u == UNROLL - 1)) group_close(m);
      }
    }
  }
  for (; b != nsafe; ++b) {
    const uint32_t oa = next_word();
    const uint32_t ob = next_word();
    uint32_t e, o;
    gather_pair<DPP>(oa, ob, lane, e, o);
    consume_pair<MOMENTS, false, NT>(e, o, (b << 7) + poff, n, out, m);
    if (MOMENTS) group_close(m);
  }
  for (; b != nblk; ++b) {
    const uint32_t oa = next_word();
    const uint32_t ob = next_word();
    uint32_t e, o;
    gather_pair<DPP>(oa, ob, lane, e, o);
    consume_pair<MOMENTS, true, NT>(e, o, (b << 7) + poff, n, out, m);
    if (MOMENTS) group_close(m);
  }
  // Tail: rw (even, < 128) more words.
  uint32_t p0 = g.prev, c0 = g.cur, xl = 0u, rem = 0u;
  if (rw) {
    uint32_t oa, ob = 0u;
    if (rw <= 64u) {
      p0 = g.prev;
      c0 = g.cur;
      xl = ring_step(g, lane0);
      oa = xl + temper_weyl(wbase + wlane);
      rem = rw & 63u;               // rw == 64 completes the chunk
      if (!rem) { p0 = g.prev; c0 = g.cur; }
    } else {
      const uint32_t xa = ring_step(g, lane0);
      oa = xa + temper_weyl(wbase + wlane);
      wbase += kChunkOmega;
      p0 = g.prev;
      c0 = g.cur;
      xl = ring_step(g, lane0);
      ob = xl + temper_weyl(wbase + wlane);
      rem = rw - 64u;
    }
    uint32_t e, o;
    gather_pair<DPP>(oa, ob, lane, e, o);
    if (poff < rw) consume_pair<MOMENTS, true, NT>(e, o, (nblk << 7) + poff, n, out, m);
    if (MOMENTS) group_close(m);
  }
  end(p0, c0, xl, rem, w_start + (uint32_t)words * kOmega, pos + words, lane);
  if constexpr (MOMENTS) {
    // The lanes' compensated sums are folded and reduced across the
    // wavefront in FP64, then rounded once to FP32: the reduction then adds
    // well under one FP32 rounding to the error of the sums.
    double v1 = (double)m.s1 - (double)m.c1, v2 = (double)m.s2 - (double)m.c2;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      v1 += __shfl_xor(v1, off);
      v2 += __shfl_xor(v2, off);
    }
    if (lane == 0) {
      sums[0] = (float)v1;
      sums[1] = (float)v2;
    }
  }
}

template <bool MOMENTS, int UNROLL, bool DPP>
__device__ __forceinline__ void serve_normals(uint32_t *st, uint64_t n, float *__restrict__ out,
                                              float *__restrict__ sums) {
  serve_normals_from<MOMENTS, UNROLL, DPP>(load_state(st), n, out, sums, ToMemory{st});
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------


// Seeds one stream per wavefront: ring and Weyl start from SplitMix64(seed + i),
// zero-ring guard, then 512 = 8 chunks of discarded steps.
__global__ __launch_bounds__(256) void k_init(uint32_t *__restrict__ state, uint64_t num_streams,
                                              uint64_t seed) {
  const uint64_t wid = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (wid >= num_streams) return;
  const uint32_t lane = lane_id();
  const uint64_t s = seed + wid;
  uint32_t lo = (uint32_t)(splitmix64_at(s, lane + 1u) >> 32);    // x_{-128+j}
  uint32_t hi = (uint32_t)(splitmix64_at(s, lane + 65u) >> 32);   // x_{-64+j}
  const uint32_t w0 = (uint32_t)(splitmix64_at(s, 129u) >> 32);   // W
  const bool any = __any((lo | hi) != 0u);
  if (!any && lane == 63u) hi = 1u;                                // x_{-1} = 1
  Ring g = ring_from(lo, hi);
  const bool lane0 = lane == 0;
#pragma unroll
  for (int c = 0; c < 8; ++c) (void)ring_step(g, lane0);
  uint32_t *st = state + wid * kStateWords;
  store_ring(st, g.prev, g.cur, 0u, 0u, lane);
  store_weyl_pos(st, w0 + 512u * kOmega, 0ull, lane);
}

// DPP (normals and moments): the pair gather without LDS.
template <uint32_t KIND, int UNROLL, bool WIDE, bool DPP = false>
__global__ __launch_bounds__(1024) void k_generate(uint32_t *__restrict__ state, uint64_t first,
                                                   uint64_t count, uint64_t n, void *__restrict__ out) {
  // Stream-major rows: each XCD takes a contiguous range of streams (measured
  // a few per cent faster than the plain order for this layout).
  const uint64_t wid = ((uint64_t)xcd_block() * blockDim.x + threadIdx.x) >> 6;
  if (wid >= count) return;
  uint32_t *st = state + (first + wid) * kStateWords;
  if constexpr (KIND == kU32 || KIND == kF32) {
    constexpr bool kPaced = KIND == kU32 && UNROLL == 2 && !WIDE;  // see emit_word
    serve_words<KIND, UNROLL, WIDE, kPaced>(st, n, reinterpret_cast<uint32_t *>(out) + wid * n);
  } else if constexpr (KIND == kNormal) {
    serve_normals<false, UNROLL, DPP>(st, n, reinterpret_cast<float *>(out) + wid * n, nullptr);
  } else {
    serve_normals<true, UNROLL, DPP>(st, n, nullptr, reinterpret_cast<float *>(out) + 2 * wid);
  }
}

// The same with cached stores, for rows that start inside a cache line and for
// words with two or more wavefronts per SIMD (cached_stores in xg_shape.h).
template <uint32_t KIND, bool DPP = false>
__global__ __launch_bounds__(1024) void k_rows_cached(uint32_t *__restrict__ state, uint64_t first, uint64_t count,
                                                      uint64_t n, uint32_t *__restrict__ out) {
  const uint64_t wid = ((uint64_t)xcd_block() * blockDim.x + threadIdx.x) >> 6;
  if (wid >= count) return;
  uint32_t *st = state + (first + wid) * kStateWords;
  if constexpr (KIND == kNormal) {
    serve_normals_from<false, 8, DPP, false>(load_state(st), n, reinterpret_cast<float *>(out) + wid * n, nullptr, ToMemory{st});
  } else {
    serve_words_from<KIND, 8, false, false, false>(load_state(st), n, out + wid * n, ToMemory{st});
  }
}

// Bulk-fill layout (see serve_words_fill): uint32 / FP32 only.
template <uint32_t KIND, int UNROLL>
__global__ __launch_bounds__(1024) void k_fill(uint32_t *__restrict__ state, uint64_t first,
                                               uint64_t count, uint64_t n, uint32_t *__restrict__ out) {
  // Plain block order: consecutive blocks (streams, hence adjacent 256-byte
  // pieces of the dense output front) land on different XCDs, which spreads
  // every XCD's writes over the whole front.  Measured faster than giving
  // each XCD a contiguous range (xcd_block) for this layout.
  const uint64_t wid = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (wid >= count) return;
  serve_words_fill<KIND, UNROLL>(state + (first + wid) * kStateWords, n, wid, count, out);
}

// ---------------------------------------------------------------------------
// skip: advance a stream by J words without producing them.
// ---------------------------------------------------------------------------

// By stepping: the recurrence runs J words and only the state is kept.
__device__ __forceinline__ void skip_by_stepping(uint32_t *st, uint64_t J) {
  WordStream s = open_stream(st);
  const uint64_t nfull = J >> 6;
  const uint32_t rem = (uint32_t)(J & 63u);
  for (uint64_t c = 0; c != nfull; ++c) (void)ring_step(s.g, s.lane0);
  const uint32_t p0 = s.g.prev, c0 = s.g.cur;
  uint32_t x = 0u;
  if (rem) x = ring_step(s.g, s.lane0);
  store_ring(st, p0, c0, x, rem, s.lane);
  store_weyl_pos(st, s.w_start + (uint32_t)J * kOmega, s.pos + J, s.lane);
}

// By jumping (xg_jump_mm.h): n = 4096, r = 128 words of 32 bits, so the
// continuation has 66 blocks of 64 words and the result four tiles of 32.
constexpr uint32_t kJumpWords = 128;               // words of z^J mod P
constexpr uint32_t kJumpBlocks = (4096 + 128) / 64;

// Wavefronts of a workgroup that shares one jump.
constexpr uint32_t kJumpWaves = 8;  // four took 8.0 us for one stream, eight take 5.9 (VALU window sums: 11.2)
constexpr uint32_t kJumpBlocksPerCu = 2;           // such workgroups that a compute unit runs at once
constexpr int kJumpQ0 = -3;                        // G's first q (tile 3 of block 0)
constexpr uint32_t kJumpQs = 2 * kJumpBlocks - kJumpQ0;

struct JumpLds {
  uint32_t s[64 * kJumpBlocks];          // the continuation's words
  uint32_t g[kJumpWords];
  uint32_t rows[32 * kJumpQs];           // toeplitz_word(q, row_word(rho)) at 32 (q - kJumpQ0) + rho
  uint32_t part[kJumpWaves][kJumpWords];  // each wavefront's share of the result
};

// One jump by a workgroup of kJumpWaves wavefronts, for launches where
// latency counts.  Wavefront 0 runs the 64 dependent steps of the
// continuation (1.6 us) while the others lay out G's rows; then each
// wavefront takes a run of consecutive blocks, all four tiles of them (tiles 2
// and 3 of a block are tiles 0 and 1 of the block before, so a block needs two
// new fragments of G and one of s), and the shares are added as words.  s is
// the stream's state on every wavefront and h_lo, h_hi the polynomial's 64-bit
// word of the lane's index.  Returns word threadIdx.x of the jumped ring (wavefronts 0
// and 1; zero elsewhere).  Every thread of the workgroup calls it.
__device__ __forceinline__ uint32_t jump_ring_wg(const StreamState &s, uint32_t h_lo, uint32_t h_hi, JumpLds &lds,
                                                 uint32_t wave) {
  const uint32_t lane = lane_id();
  __syncthreads();  // an earlier jump's reads of lds are done
  if (wave == 1) {
    lds.g[2 * lane] = h_lo;
    lds.g[2 * lane + 1] = h_hi;
  }
  __syncthreads();
  if (wave == 0) {
    const bool lane0 = lane == 0;
    lds.s[lane] = s.prev;
    lds.s[64 + lane] = s.cur;
    Ring r = ring_from(s.prev, s.cur);
#pragma unroll 4
    for (uint32_t c = 2; c < kJumpBlocks; ++c) lds.s[64 * c + lane] = ring_step(r, lane0);
  } else {
    for (uint32_t i = threadIdx.x - 64; i < 32 * kJumpQs; i += 64 * (kJumpWaves - 1))
      lds.rows[i] = dev::toeplitz_word(lds.g, kJumpWords, (int)(i / 32) + kJumpQ0, dev::row_word(i % 32));
  }
  __syncthreads();
  const dev::TransposeLane tl = dev::transpose_lane(lane);
  constexpr uint32_t kEach = kJumpBlocks / kJumpWaves, kMore = kJumpBlocks % kJumpWaves;  // the last kMore take one more
  const uint32_t late = wave > kJumpWaves - kMore ? wave - (kJumpWaves - kMore) : 0u;
  const uint32_t c0 = kEach * wave + late;
  // Tile t of block c: q = 2 c - t + h.
  const uint32_t *rows = lds.rows + 32 * (2 * c0 - kJumpQ0) + lane;
  dev::tile_t acc[4] = {};
  dev::frag_t a2 = dev::frag(dev::one_bits(rows[-64])), a3 = dev::frag(dev::one_bits(rows[-96]));
  auto block = [&](uint32_t c) {
    const dev::frag_t b = dev::frag(dev::half_bits(dev::word_bits(lds.s[64 * c + lane], tl)));
    const dev::frag_t a0 = dev::frag(dev::one_bits(rows[0])), a1 = dev::frag(dev::one_bits(rows[-32]));
    acc[0] = dev::mm_step(a0, b, acc[0]);
    acc[1] = dev::mm_step(a1, b, acc[1]);
    acc[2] = dev::mm_step(a2, b, acc[2]);
    acc[3] = dev::mm_step(a3, b, acc[3]);
    a2 = a0;
    a3 = a1;
    rows += 64;
  };
#pragma unroll
  for (uint32_t i = 0; i < kEach; ++i) block(c0 + i);
  if (wave >= kJumpWaves - kMore) block(c0 + kEach);
  lds.part[wave][lane] = dev::tile_words(acc[0], acc[1], tl);
  lds.part[wave][64 + lane] = dev::tile_words(acc[2], acc[3], tl);
  __syncthreads();
  uint32_t y = 0;
  if (wave < 2) {
#pragma unroll
    for (uint32_t w = 0; w < kJumpWaves; ++w) y ^= lds.part[w][threadIdx.x];
  }
  return y;
}

__device__ __forceinline__ void jump_weyl(StreamState &s, uint64_t J) {
  s.weyl += (uint32_t)J * kOmega;
  s.pos += J;
}

// Few streams: one workgroup each.
__global__ __launch_bounds__(kJumpWaves * 64, 4) void k_skip_wg(uint32_t *__restrict__ state, uint64_t first, uint64_t J,
                                                             JumpPoly g) {
  __shared__ JumpLds lds;
  const uint32_t lane = lane_id();
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  uint32_t *st = state + (first + blockIdx.x) * kStateWords;
  StreamState s = load_state(st);
  const uint64_t h = g.w[lane];
  const uint32_t y = jump_ring_wg(s, (uint32_t)h, (uint32_t)(h >> 32), lds, wave);
  jump_weyl(s, J);
  if (wave < 2) st[threadIdx.x] = y;
  if (wave == 0) store_weyl_pos(st, s.weyl, s.pos, lane);
}

// Many streams by one J: a wavefront per stream, with G's fragments laid out
// once per workgroup in LDS, 16 bytes per lane (tiles 2 and 3 of a block are
// tiles 0 and 1 of the block before).  Per 64 words a wavefront spends about
// 35 VALU instructions (step, bit transpose, expansion; some 110 cycles) beside
// four matrix instructions (4 x 32 cycles); with four wavefronts per SIMD the
// two together take 205 cycles.  4096 streams: 28 us, 65536: 392 us (70 and
// 951 us with the window sums on the VALU).
constexpr uint32_t kSkipWaves = 8;
constexpr uint32_t kSkipQs = 2 * kJumpBlocks + 3;  // q from -1, and a block more than is used

__global__ __launch_bounds__(kSkipWaves * 64, 4) void k_skip_many(uint32_t *__restrict__ state, uint64_t first,
                                                               uint64_t count, uint64_t J, JumpPoly g) {
  __shared__ uint4 frags[32 * kSkipQs];
  __shared__ uint32_t gw[kJumpWords];
  const uint32_t lane = lane_id();
  if (threadIdx.x < 64) {
    const uint64_t h = g.w[lane];
    gw[2 * lane] = (uint32_t)h;
    gw[2 * lane + 1] = (uint32_t)(h >> 32);
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < 32 * kSkipQs; i += 64 * kSkipWaves)
    frags[i] = dev::one_bits(dev::toeplitz_word(gw, kJumpWords, (int)(i / 32) - 1, dev::row_word(i % 32)));
  __syncthreads();
  const dev::TransposeLane tl = dev::transpose_lane(lane);
  const bool lane0 = lane == 0;
  const uint64_t waves = (uint64_t)gridDim.x * kSkipWaves;
  for (uint64_t k = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; k < count; k += waves) {
    uint32_t *st = state + (first + k) * kStateWords;
    StreamState s = load_state(st);
    Ring r = ring_from(s.prev, s.cur);
    dev::tile_t acc[4] = {};
    uint4 a2 = make_uint4(0, 0, 0, 0), a3 = a2;
    const uint4 *f = frags + lane;
    uint4 a1 = f[0], a0 = f[32];  // q = 2 c - 1 + h, 2 c + h
    uint4 b = dev::half_bits(dev::word_bits(s.prev, tl));
    // Each trip multiplies block c while it prepares block c + 1 (x: its
    // words), so that the VALU work fills the matrix instructions' time.
    auto block = [&](uint32_t x) {
      f += 64;
      const uint4 n1 = f[0], n0 = f[32];
      acc[0] = dev::mm_step(dev::frag(a0), dev::frag(b), acc[0]);
      acc[1] = dev::mm_step(dev::frag(a1), dev::frag(b), acc[1]);
      acc[2] = dev::mm_step(dev::frag(a2), dev::frag(b), acc[2]);
      acc[3] = dev::mm_step(dev::frag(a3), dev::frag(b), acc[3]);
      const uint4 bn = dev::half_bits(dev::word_bits(x, tl));
      a2 = a0;
      a3 = a1;
      a0 = n0;
      a1 = n1;
      b = bn;
    };
    block(s.cur);
#pragma unroll 2
    for (uint32_t c = 2; c < kJumpBlocks; ++c) block(ring_step(r, lane0));
    block(0u);
    jump_weyl(s, J);
    st[lane] = dev::tile_words(acc[0], acc[1], tl);
    st[64 + lane] = dev::tile_words(acc[2], acc[3], tl);
    store_weyl_pos(st, s.weyl, s.pos, lane);
  }
}

__global__ __launch_bounds__(256) void k_skip_steps(uint32_t *__restrict__ state, uint64_t first, uint64_t count,
                                                    uint64_t J) {
  const uint64_t wid = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (wid >= count) return;
  skip_by_stepping(state + (first + wid) * kStateWords, J);
}

// ---------------------------------------------------------------------------
// Rows cut into parts (xg_split.h): launches of few streams.
// ---------------------------------------------------------------------------
// Where part k of the launch's i-th stream keeps its start state: word t at
// out[i row + k part + (t / 64) chunk + t % 64], i.e. in the part's own first
// three chunks in either layout (a part has at least four).
struct SplitPlaces {
  uint64_t row, part, chunk;
};

// Start states of all parts: workgroup b jumps stream b % count by
// (b / count) 2^exp words (part 0: a copy) and leaves ring, Weyl value and
// position in the part's place in the output.  Nothing else reads the streams'
// states after this kernel, so k_split_* may write them back.
__global__ __launch_bounds__(kJumpWaves * 64, 4) void k_split_starts(const uint32_t *__restrict__ state, uint64_t first,
                                                                  uint32_t count, uint32_t exp,
                                                                  const uint64_t *__restrict__ table,
                                                                  uint32_t *__restrict__ out, SplitPlaces at) {
  __shared__ JumpLds lds;
  const uint32_t lane = lane_id();
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t k = blockIdx.x / count, i = blockIdx.x % count;
  StreamState s = load_state(state + (first + i) * kStateWords);
  uint32_t *o = out + i * at.row + k * at.part;
  if (k) {
    const uint64_t h = table[(uint64_t)split_entry(exp, k) * 64 + lane];
    const uint32_t y = jump_ring_wg(s, (uint32_t)h, (uint32_t)(h >> 32), lds, wave);
    jump_weyl(s, (uint64_t)k << exp);
    if (wave < 2) o[wave * at.chunk + lane] = y;
  } else if (wave < 2) {
    o[wave * at.chunk + lane] = wave ? s.cur : s.prev;
  }
  if (wave == 0 && lane < 3u) o[2 * at.chunk + lane] = lane == 0 ? s.weyl : (uint32_t)(s.pos >> (32u * (lane - 1u)));
}

__device__ __forceinline__ StreamState load_split(const uint32_t *o, uint64_t chunk) {
  const uint32_t lane = lane_id();
  StreamState s;
  s.prev = o[lane];
  s.cur = o[chunk + lane];
  const int v = lane < 3u ? (int)o[2 * chunk + lane] : 0;
  s.weyl = (uint32_t)__builtin_amdgcn_readlane(v, 0);
  s.pos = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(v, 1) |
          ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(v, 2) << 32);
  return s;
}

// One wavefront per part: wavefront (k, i) starts from the state in part k's
// place, writes the part's values over it (every value depends on all of the
// state, so the loads are done first), and the last part writes the stream's
// end state.
template <uint32_t KIND, bool FILL>
__global__ __launch_bounds__(256) void k_split(uint32_t *__restrict__ state, uint64_t first, uint32_t count,
                                               uint64_t n, uint32_t parts, uint32_t exp, uint32_t *out,
                                               SplitPlaces at) {
  const uint32_t wid = (uint32_t)__builtin_amdgcn_readfirstlane((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
  const uint32_t k = wid / count, i = wid % count;
  if (k >= parts) return;
  const uint64_t done = (uint64_t)k << exp;
  const bool last = k + 1 == parts;
  const uint64_t nk = last ? n - done : 1ull << exp;
  uint32_t *o = out + i * at.row + k * at.part;
  const StreamState s0 = load_split(o, at.chunk);
  uint32_t *dst = last ? state + (first + i) * kStateWords : nullptr;
  if constexpr (KIND == kNormal) {
    serve_normals_from<false, 8, true, false>(s0, nk, reinterpret_cast<float *>(o), nullptr, ToMemory{dst});
  } else if constexpr (FILL) {
    const uint32_t lane = lane_id();
    uint32_t *tail = out + (n >> 6) * at.chunk + i * (n & 63u) + lane;
    serve_chunks<KIND, 8, false>(s0, nk, o + lane, at.chunk, tail, dst);
  } else {
    serve_words_from<KIND, 8, false, false, false>(s0, nk, o, ToMemory{dst});
  }
}

// Box-Muller on caller-supplied word pairs (the same device function the
// generators use): out[2m], out[2m + 1] from words[2m], words[2m + 1].
__global__ __launch_bounds__(256) void k_box_muller(const uint32_t *__restrict__ words, uint64_t pairs,
                                                    float *__restrict__ out) {
  const uint64_t m = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= pairs) return;
  float z0, z1;
  box_muller(words[2 * m], words[2 * m + 1], z0, z1);
  out[2 * m] = z0;
  out[2 * m + 1] = z1;
}

// Workspace words of the batch kernels: work[0] the queue counter, work[1]
// the error word, work[2] the queue items (groups), work[3] the table entries.
__global__ void k_work_init(uint32_t *work, uint32_t num_groups, uint32_t num_reqs) {
  if (threadIdx.x < 64) work[threadIdx.x] = threadIdx.x == 2 ? num_groups : threadIdx.x == 3 ? num_reqs : 0u;
}

// Re-arms the queue of a table that is already in place.
__global__ void k_work_requeue(uint32_t *work) {
  if (threadIdx.x == 0) work[0] = 0u;
}

// Checks of a segment entry (kReqSegment): tile k of a longer request, whose
// start state sits in staging slot `slot`.
__device__ __forceinline__ bool seg_entry_ok(const xg_request &q, uint64_t num_streams, const SegmentArgs &seg) {
  const uint32_t k = (q.flags >> 8) & 0xFFu, slot = q.flags >> 16;
  return (q.flags & kReqSegment) && !(q.flags & kReqUndefinedBits) && q.stream < num_streams &&
         q.dtype <= XG_NORMAL && seg.stage && slot < seg.max_slots && k <= seg.max_k && (k == 0 || seg.jump_table);
}

// Start state of every segment entry of a table: its stream's state jumped by
// k L words (k = 0: a copy) into staging slot `slot`.  One wavefront per
// entry (work[3] entries); others, and entries that fail the checks, are
// skipped (the batch kernel skips those too).  The batch kernel then starts
// each segment from its slot, so no segment reads a stream state that the
// request's last segment rewrites.
__global__ __launch_bounds__(kJumpWaves * 64, 4) void k_seg_starts(const uint32_t *__restrict__ state,
                                                                uint64_t num_streams,
                                                                const xg_request *__restrict__ reqs,
                                                                const uint32_t *__restrict__ work,
                                                                SegmentArgs seg) {
  // One workgroup per segment entry (grid-stride over the table); the jump by
  // k L words is jump_ring_wg with the polynomial of table entry k - 1.
  __shared__ JumpLds lds;
  const uint32_t lane = lane_id();
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t entries = work[3];
  for (uint32_t r = blockIdx.x; r < entries; r += gridDim.x) {
    const xg_request q = reqs[r];  // the same on every thread of the workgroup
    if (!(q.flags & kReqSegment) || !seg_entry_ok(q, num_streams, seg)) continue;
    const uint32_t k = (uint32_t)__builtin_amdgcn_readfirstlane((int)((q.flags >> 8) & 0xFFu));
    const uint32_t slot = q.flags >> 16;
    StreamState s = load_state(state + q.stream * kStateWords);
    uint32_t *dst = seg.stage + (uint64_t)slot * kStateWords;
    if (k) {
      const uint64_t h = seg.jump_table[(uint64_t)(k - 1) * 64 + lane];
      const uint32_t y = jump_ring_wg(s, (uint32_t)h, (uint32_t)(h >> 32), lds, wave);
      jump_weyl(s, (uint64_t)k * seg.seg_words);
      if (wave < 2) dst[threadIdx.x] = y;
    } else if (wave < 2) {
      dst[threadIdx.x] = wave ? s.cur : s.prev;
    }
    if (wave == 0) store_weyl_pos(dst, s.weyl, s.pos, lane);
  }
}

// Persistent batched kernel (launched with no more blocks than the device
// holds at once): each wavefront serves the group of its own index, then its
// further ones, dealt or taken from an atomic queue (work[0], counting from the
// grid's wavefronts), until it passes work[2] groups; every wavefront reaches
// the exit.  A plain
// entry reads and rewrites its stream's state; a segment entry
// starts from its staged start state and only the request's last segment
// writes the stream's state.  Outputs leave through plain (cached) stores
// (emit_word).
template <int UNROLL, bool WIDE>
__global__ __launch_bounds__(1024) void k_batch(uint32_t *__restrict__ state, uint64_t num_streams,
                                                const xg_request *__restrict__ reqs,
                                                const uint32_t *__restrict__ groups, uint32_t *__restrict__ out,
                                                uint64_t out_elems, uint32_t *__restrict__ work,
                                                SegmentArgs seg) {
  const uint32_t lane = lane_id();
  const uint32_t num_groups = work[2], num_reqs = work[3];
  // Items come largest first.  A wavefront's first item is its own index in the
  // grid (the first pops would hand out exactly those items, one atomic at a
  // time); small ones after that are dealt (deal_items), and trips to the queue
  // take batch_take others from the counter, offset by the wavefronts in the
  // grid.
  const uint32_t wpb = blockDim.x >> 6;
  const uint32_t waves = gridDim.x * wpb;
  const uint32_t wave = blockIdx.x * wpb + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const bool dealt = deal_items(reqs, num_reqs, groups, num_groups, waves, 1u << 16);
  uint32_t g0 = wave;
  uint32_t take = 1, round = 0;
  for (;;) {
    if (g0 >= num_groups) break;
    const uint32_t g_end = num_groups - g0 < take ? num_groups : g0 + take;
    uint64_t served = 0;
    for (uint32_t g = g0; g < g_end; ++g) {
      const uint32_t r0 = groups[g], r1 = groups[g + 1];
      if (r0 > r1 || r1 > num_reqs) {
        if (lane == 0) atomicOr(&work[1], 1u);
        continue;
      }
      // A group's requests continue one stream, whose state stays in registers
      // between them, and the next request is loaded while one is served: both
      // chains of loads bound short requests (plan and batch of 4000 requests
      // of 2^6 to 2^10 words on 400 streams: 69 us with the state in memory, 64
      // so).
      StreamState s{};
      uint32_t *held = nullptr;  // whose state s is
      auto put_back = [&] {
        if (held) write_state(held, s.prev, s.cur, 0u, 0u, s.weyl, s.pos, lane);
        held = nullptr;
      };
      xg_request q{};
      if (r0 < r1) q = reqs[r0];
      for (uint32_t r = r0; r < r1; ++r) {
        const xg_request next = reqs[r + 1 < r1 ? r + 1 : r];  // on its way while q is served
        const bool is_seg = (q.flags & kReqSegment) != 0;
        const bool ok = (is_seg ? seg_entry_ok(q, num_streams, seg)
                                : q.stream < num_streams && q.dtype <= XG_NORMAL && q.flags == 0u) &&
                        q.out_offset <= out_elems && q.n <= out_elems - q.out_offset;
        if (ok) {
          uint32_t *st = state + q.stream * kStateWords;
          if (is_seg || st != held) {
            put_back();
            s = load_state(is_seg ? seg.stage + (uint64_t)(q.flags >> 16) * kStateWords : st);
          }
          held = !is_seg || (q.flags & kReqLast) ? st : nullptr;
          uint32_t *o = out + q.out_offset;
          const StreamState s0 = s;
          if (q.dtype == XG_U32) {
            serve_words_from<kU32, UNROLL, WIDE, false, false>(s0, q.n, o, ToRegisters{&s});
          } else if (q.dtype == XG_F32) {
            serve_words_from<kF32, UNROLL, WIDE, false, false>(s0, q.n, o, ToRegisters{&s});
          } else {
            serve_normals_from<false, UNROLL, true, false>(s0, q.n, reinterpret_cast<float *>(o), nullptr,
                                                           ToRegisters{&s});
          }
          served += q.n;
        } else if (lane == 0) {
          atomicOr(&work[1], 1u);
        }
        q = next;
      }
      put_back();
    }
    if (dealt) {
      g0 = dealt_item(++round, wave, waves, num_groups);
      continue;
    }
    take = batch_take(served, g_end - g0, g0, num_groups, waves);
    uint32_t c = 0;
    if (lane == 0) c = atomicAdd(&work[0], take);
    g0 = waves + (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
  }
}

template <uint32_t KIND>
hipError_t launch_generate_k(const Shape &sh, dim3 grid, dim3 block, uint32_t *state, uint64_t first,
                             uint64_t count, uint64_t n, void *out, int num_cus, hipStream_t stream) {
  hipError_t e = hipSuccess;
  constexpr bool kWords = KIND == kU32 || KIND == kF32;
  if constexpr (!kWords) {
    // Normals with at most one wavefront per SIMD: the DPP pair gather.
    if (count <= 4u * (uint64_t)(num_cus > 0 ? num_cus : 1)) {
      switch (sh.unroll) {
        case 1: return launch((k_generate<KIND, 1, false, true>), grid, block, 0, stream, state, first, count, n, out);
        case 2: return launch((k_generate<KIND, 2, false, true>), grid, block, 0, stream, state, first, count, n, out);
        case 4: return launch((k_generate<KIND, 4, false, true>), grid, block, 0, stream, state, first, count, n, out);
        default: return launch((k_generate<KIND, 8, false, true>), grid, block, 0, stream, state, first, count, n, out);
      }
    }
  }
  const bool wide = kWords && sh.store_words == 4;
  const size_t lds = wide ? (size_t)sh.waves_per_block * 1024u : 0u;
  if (wide) {
    if (sh.unroll == 4) {
      e = launch((k_generate<KIND, 4, kWords>), grid, block, lds, stream, state, first, count, n, out);
    } else {
      e = launch((k_generate<KIND, 8, kWords>), grid, block, lds, stream, state, first, count, n, out);
    }
    return e;
  }
  const size_t stage = kWords ? 0u : (size_t)sh.waves_per_block * 2048u;  // normals_stage
  switch (sh.unroll) {
    case 1: e = launch((k_generate<KIND, 1, false>), grid, block, stage, stream, state, first, count, n, out); break;
    case 2: e = launch((k_generate<KIND, 2, false>), grid, block, stage, stream, state, first, count, n, out); break;
    case 4: e = launch((k_generate<KIND, 4, false>), grid, block, stage, stream, state, first, count, n, out); break;
    default: e = launch((k_generate<KIND, 8, false>), grid, block, stage, stream, state, first, count, n, out); break;
  }
  return e;
}

}  // namespace

uint32_t auto_waves_per_block(uint64_t count, int num_cus) {
  return count >= 4 * (uint64_t)(num_cus > 0 ? num_cus : 1) ? 4 : 1;
}

bool shape_valid(const Shape &s) {
  const bool wpb = s.waves_per_block == 1 || s.waves_per_block == 2 || s.waves_per_block == 4 ||
                   s.waves_per_block == 8 || s.waves_per_block == 16;
  const bool un = s.unroll == 1 || s.unroll == 2 || s.unroll == 4 || s.unroll == 8;
  const bool sw = s.store_words == 1 || (s.store_words == 4 && s.unroll >= 4);
  return wpb && un && sw && s.blocks_per_cu >= 1 && s.blocks_per_cu <= 32;
}

hipError_t launch_init(uint32_t *state, uint64_t num_streams, uint64_t seed, hipStream_t stream) {
  hipError_t e = hipSuccess;
  const uint64_t blocks = (num_streams + 3) / 4;
  e = launch(k_init, dim3((uint32_t)blocks), dim3(256), 0, stream, state, num_streams, seed);
  return e;
}

hipError_t launch_fill(Kind kind, const Shape &shape, uint32_t *state, uint64_t first, uint64_t count,
                       uint64_t n, uint32_t *out, hipStream_t stream) {
  hipError_t e = hipSuccess;
  const uint64_t wpb = shape.waves_per_block;
  const dim3 grid((uint32_t)((count + wpb - 1) / wpb));
  const dim3 block((uint32_t)(wpb * kWave));
  const bool f = kind == kF32;
  switch (shape.unroll) {
    case 1: if (f) e = launch((k_fill<kF32, 1>), grid, block, 0, stream, state, first, count, n, out);
            else e = launch((k_fill<kU32, 1>), grid, block, 0, stream, state, first, count, n, out);
            break;
    case 2: if (f) e = launch((k_fill<kF32, 2>), grid, block, 0, stream, state, first, count, n, out);
            else e = launch((k_fill<kU32, 2>), grid, block, 0, stream, state, first, count, n, out);
            break;
    case 4: if (f) e = launch((k_fill<kF32, 4>), grid, block, 0, stream, state, first, count, n, out);
            else e = launch((k_fill<kU32, 4>), grid, block, 0, stream, state, first, count, n, out);
            break;
    default: if (f) e = launch((k_fill<kF32, 8>), grid, block, 0, stream, state, first, count, n, out);
             else e = launch((k_fill<kU32, 8>), grid, block, 0, stream, state, first, count, n, out);
             break;
  }
  return e;
}

hipError_t launch_box_muller(const uint32_t *words, uint64_t pairs, float *out, hipStream_t stream) {
  hipError_t e = hipSuccess;
  e = launch(k_box_muller, dim3((uint32_t)((pairs + 255) / 256)), dim3(256), 0, stream, words, pairs, out);
  return e;
}

hipError_t launch_skip(uint32_t *state, uint64_t first, uint64_t count, uint64_t J, const JumpPoly *g,
                       int num_cus, hipStream_t stream) {
  const uint64_t cus = num_cus > 0 ? (uint64_t)num_cus : 1;
  if (!g)
    return launch(k_skip_steps, dim3((uint32_t)((count + 3) / 4)), dim3(256), 0, stream, state, first, count, J);
  // Up to four streams per compute unit a workgroup each (7.0 us up to one, 9
  // up to two, 12.7 up to three, 16.0 at four), beyond that a wavefront each
  // (16.8 us up to eight, 30 us at sixteen).
  if (count <= 4 * cus)
    return launch(k_skip_wg, dim3((uint32_t)count), dim3(kJumpWaves * 64), 0, stream, state, first, J, *g);
  const uint64_t blocks = (count + kSkipWaves - 1) / kSkipWaves;
  return launch(k_skip_many, dim3((uint32_t)(blocks < 2 * cus ? blocks : 2 * cus)), dim3(kSkipWaves * 64), 0, stream,
                state, first, count, J, *g);
}

hipError_t launch_generate(Kind kind, const Shape &shape, uint32_t *state, uint64_t first,
                           uint64_t count, uint64_t n, void *out, int num_cus, hipStream_t stream) {
  const uint64_t wpb = shape.waves_per_block;
  const dim3 grid((uint32_t)((count + wpb - 1) / wpb));
  const dim3 block((uint32_t)(wpb * kWave));
  switch (kind) {
    case kU32: return launch_generate_k<kU32>(shape, grid, block, state, first, count, n, out, num_cus, stream);
    case kF32: return launch_generate_k<kF32>(shape, grid, block, state, first, count, n, out, num_cus, stream);
    case kNormal:
      return launch_generate_k<kNormal>(shape, grid, block, state, first, count, n, out, num_cus, stream);
    default: return launch_generate_k<kMoments>(shape, grid, block, state, first, count, n, out, num_cus, stream);
  }
}

hipError_t launch_split(Kind kind, bool fill, const Split &sp, uint32_t *state, uint64_t first, uint64_t count,
                        uint64_t n, const uint64_t *table, void *out, int num_cus, hipStream_t stream) {
  const uint64_t waves = count * sp.parts;
  const uint64_t wpb = auto_waves_per_block(waves, num_cus);
  uint32_t *o = static_cast<uint32_t *>(out);
  const uint64_t part = 1ull << sp.exp;
  const SplitPlaces at = fill ? SplitPlaces{64, part * count, 64 * count} : SplitPlaces{n, part, 64};
  hipError_t e = launch(k_split_starts, dim3((uint32_t)waves), dim3(kJumpWaves * 64), 0, stream, state, first, count,
                        sp.exp, table, o, at);
  if (e != hipSuccess) return e;
  auto run = [&](auto kernel) {
    return launch(kernel, dim3((uint32_t)((waves + wpb - 1) / wpb)), dim3((uint32_t)(wpb * kWave)), 0, stream, state,
                  first, count, n, sp.parts, sp.exp, o, at);
  };
  if (kind == kNormal) return run(k_split<kNormal, false>);
  if (kind == kF32) return fill ? run(k_split<kF32, true>) : run(k_split<kF32, false>);
  return fill ? run(k_split<kU32, true>) : run(k_split<kU32, false>);
}

hipError_t launch_rows_cached(Kind kind, uint32_t waves_per_block, uint32_t *state, uint64_t first, uint64_t count,
                              uint64_t n, void *out, int num_cus, hipStream_t stream) {
  const uint64_t wpb = waves_per_block;
  auto run = [&](auto kernel) {
    return launch(kernel, dim3((uint32_t)((count + wpb - 1) / wpb)), dim3((uint32_t)(wpb * kWave)),
                  kind == kNormal ? wpb * 2048 : 0, stream, state, first, count, n, static_cast<uint32_t *>(out));
  };
  if (kind == kU32) return run(k_rows_cached<kU32>);
  if (kind == kF32) return run(k_rows_cached<kF32>);
  // Normals: the pair gather as for launch_generate.
  const bool dpp = count <= 4u * (uint64_t)(num_cus > 0 ? num_cus : 1);
  return dpp ? run(k_rows_cached<kNormal, true>) : run(k_rows_cached<kNormal, false>);
}

hipError_t launch_work_init(uint32_t *work, uint32_t num_groups, uint32_t num_reqs, hipStream_t stream) {
  return launch(k_work_init, dim3(1), dim3(64), 0, stream, work, num_groups, num_reqs);
}

hipError_t launch_work_requeue(uint32_t *work, hipStream_t stream) {
  return launch(k_work_requeue, dim3(1), dim3(64), 0, stream, work);
}

hipError_t launch_seg_starts(const uint32_t *state, uint64_t num_streams, const xg_request *reqs,
                             uint32_t max_entries, const uint32_t *work, const SegmentArgs &seg, int num_cus,
                             hipStream_t stream) {
  if (max_entries == 0) return hipSuccess;
  // As many workgroups as fit on the chip at once, each taking every
  // gridDim-th entry.
  const uint32_t slots = (num_cus > 0 ? (uint32_t)num_cus : 1u) * kJumpBlocksPerCu;
  const uint32_t blocks = max_entries < slots ? max_entries : slots;
  return launch(k_seg_starts, dim3(blocks), dim3(kJumpWaves * 64), 0, stream, state, num_streams, reqs, work, seg);
}

hipError_t launch_batch(const Shape &shape, int num_cus, uint32_t *state, uint64_t num_streams,
                        const xg_request *reqs, const uint32_t *groups, uint32_t max_groups, uint32_t *out,
                        uint64_t out_elems, uint32_t *work, hipStream_t stream, const SegmentArgs *seg) {
  uint64_t blocks = (uint64_t)(num_cus > 0 ? num_cus : 1) * shape.blocks_per_cu;
  const uint64_t need = ((uint64_t)max_groups + shape.waves_per_block - 1) / shape.waves_per_block;
  if (need < blocks) blocks = need ? need : 1;
  const dim3 block(shape.waves_per_block * kWave);
  const size_t lds = shape.store_words == 4 ? (size_t)shape.waves_per_block * 1024u : 0u;  // wide-store staging
  SegmentArgs sa{};
  if (seg) sa = *seg;
  auto run = [&](auto kernel) {
    return launch_persistent(kernel, blocks, block, lds, num_cus, stream, state, num_streams, reqs, groups, out,
                             out_elems, work, sa);
  };
  if (shape.store_words == 4) return shape.unroll == 4 ? run(k_batch<4, true>) : run(k_batch<8, true>);
  switch (shape.unroll) {
    case 1: return run(k_batch<1, false>);
    case 2: return run(k_batch<2, false>);
    case 4: return run(k_batch<4, false>);
    default: return run(k_batch<8, false>);
  }
}

}  // namespace xg
