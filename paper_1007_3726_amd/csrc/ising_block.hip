// Several sweeps per launch on rows held in LDS.
//
// A lone lattice of up to a few thousand squared, or a batch of them, has
// too little work per colour step for a launch of its own: a launch costs
// 5 us whatever it does (the launch itself, the loads, one lane's chain of
// sixteen Philox blocks), 512^2 has 0.05 us of arithmetic in it.
// Here a workgroup takes a strip of rows of one lattice with H = 2 K halo
// rows above and below into LDS, runs K sweeps on them with block barriers
// between the colour steps, and writes its own rows back.  Each colour step
// the rows that are still valid shrink by one at either end (their outer
// neighbours were not updated), so after 2 K steps exactly the strip's own
// rows are left: the halo rows are computed twice (by this strip and by the
// one that owns them) with the same uniforms, which is what the launches
// saved pay for.  Strips read one copy of the planes and write another, so
// no workgroup waits for another one.  A lattice of one strip needs no
// halo: its rows wrap and all n sweeps run in one launch.
//
// The unit of work is a 32-bit half of a word: its eight Philox blocks are
// split over ls = 1, 2, 4 or 8 adjacent lanes, so that few rows still make
// enough waves for the compute unit's four SIMDs.  Every lane of a half
// decides its own sites and the flips are OR-ed over the half's lanes (DPP
// within eight lanes).
//
// E/M: counted over the strip's own rows after each colour-1 step, summed
// per wave, then in LDS; a single strip writes (E, M) itself, several strips
// leave partials that the next launch (or launch_block_finalize after the
// last) reduces.
//
// Bound by the instructions of one workgroup's steps (halves computed in
// halos included) plus 5 us per launch.  Measured, us per sweep with the
// (E, M) series, a launch per colour step (or the LDS kernel that this one
// replaced) before: 64^2 4.29 -> 0.90, 512^2 10.3 -> 2.5, 1002^2 16.6 -> 3.9,
// 4096^2 11.7 -> 10.3; 24 lattices of 8^2 to 64^2 8.95 -> 1.01.
//
// The paper's generators and pools run in the same blocks.  A word's
// generator is affine in its steps, so every lane of a half jumps to its own
// values, and the halo rows' generators need no second copy: a strip advances
// them from the states before the call, and one last kernel advances the
// caller's.  A pool's patterns are read from memory, several rows ahead.
// us per sweep before -> after, LCG / linear pool / random pool: 64^2 9.0 / 8.4
// / 8.6 -> 0.73 / 0.99 / 1.0; 1024^2 9.7 / 9.7 / 10.9 -> 2.9 / 2.8 / 3.7;
// 4096^2 10.6 / 9.7 / 12.2 -> 6.7 / 3.7 / 8.8; 16384^2 linear 28.3 -> 16.1.
#include <algorithm>
#include <cstring>

#include "ising_batch.hpp"
#include "ising_block.hpp"
#include "ising_runtime.hpp"

#if defined(__HIP_DEVICE_COMPILE__)
#define ISING_CONSTANT_AS __attribute__((address_space(4)))
#else
#define ISING_CONSTANT_AS
#endif

namespace ising {
namespace {

// Sweeps done before launch j of m that share n sweeps.
__device__ __forceinline__ int64_t sweeps_before(int64_t n, int64_t j, int64_t m) {
  const int64_t each = n / m, more = n - each * m;  // the first `more` launches take one more
  return each * j + (j < more ? j : more);
}

template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, ROWS == 0xf);
}

// OR over groups of LS adjacent lanes, in every lane.
template <int LS>
__device__ __forceinline__ uint32_t lanes_or(uint32_t v) {
  if (LS >= 2) v |= dpp<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  if (LS >= 4) v |= dpp<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  if (LS >= 8) v |= dpp<0x141>(v);  // row_half_mirror
  return v;
}

// Sum over the wave, in lane 63.
__device__ __forceinline__ uint32_t wave_total(uint32_t v) {
  v += dpp<0x111>(v);
  v += dpp<0x112>(v);
  v += dpp<0x114>(v);
  v += dpp<0x118>(v);
  v += dpp<0x142, 0xa>(v);
  v += dpp<0x143, 0xc>(v);
  return v;
}

// How a half's uniforms are drawn: rows of whole Philox blocks (L % 8 == 0)
// with the plain compares or the cut, or rows that start anywhere in a block.
// kLcg: the word's generator; kPool, kPoolLinear: patterns.
enum { kCompare = 0, kCut = 1, kAnyRow = 2, kAnyRowCut = 3, kLcg = 4, kPool = 5, kPoolLinear = 6 };

// Random planes of this lane's 32 / LS sites of a half, at their places in
// the half (bits of other lanes' sites mean nothing).  `at`: colour-local
// index of the lane's first site, over 4 where rows are whole blocks.
template <int LS, int MODE, bool SERIAL>
__device__ __forceinline__ void half_planes(uint32_t at, int sub, uint32_t k0, uint32_t k1,
                                            uint32_t t, uint32_t ctr3, uint32_t t4, uint32_t t8,
                                            uint32_t cut_x, uint64_t cut_c, uint32_t& a,
                                            uint32_t& b) {
  constexpr int NB = 8 / LS;
  a = b = 0;
  if (MODE == kCut) {
    uint32_t acc[4] = {0, 0, 0, 0};
    cut_blocks<0, NB - 1, SERIAL>(acc, (uint64_t)kM0 * at, 0, k0, k1, t, ctr3, cut_x, cut_c);
    cut_planes(acc, a, b);
  } else if (MODE == kCompare) {
#pragma unroll
    for (int q = NB - 1; q >= 0; --q) {
      uint32_t x0 = at + (uint32_t)q, x1 = 0, x2 = t, x3 = ctr3;
      if (SERIAL) asm("" : "+v"(x0), "+v"(a), "+v"(b));
      philox4x32_10(x0, x1, x2, x3, k0, k1);
      shift_in4(a, b, x0, x1, x2, x3, t4, t8);
    }
  } else {
    // NB + 1 blocks cover the sites; the first block's r lowest outputs
    // belong to the sites before
    const uint32_t g = at >> 2, r = at & 3u;
    if (MODE == kAnyRowCut) {
      uint32_t acc[4] = {0, 0, 0, 0};
      cut_blocks<1, NB - 1, SERIAL>(acc, (uint64_t)kM0 * g, 0, k0, k1, t, ctr3, cut_x, cut_c);
      cut_planes(acc, a, b);
    } else {
      for (int q = NB; q >= 1; --q) {
        uint32_t x0 = g + (uint32_t)q, x1 = 0, x2 = t, x3 = ctr3;
        if (SERIAL) asm("" : "+v"(x0), "+v"(a), "+v"(b));
        philox4x32_10(x0, x1, x2, x3, k0, k1);
        shift_in4(a, b, x0, x1, x2, x3, t4, t8);
      }
    }
    uint32_t x0 = g, x1 = 0, x2 = t, x3 = ctr3, a0 = 0, b0 = 0;
    if (SERIAL) asm("" : "+v"(x0), "+v"(a), "+v"(b));
    philox4x32_10(x0, x1, x2, x3, k0, k1);
    shift_in4(a0, b0, x0, x1, x2, x3, t4, t8);
    if (MODE == kAnyRowCut) {  // (r4, r8) -> (up, low)
      a0 ^= 15u;
      b0 ^= 15u;
    }
    a = (a << (4u - r)) | (a0 >> r);
    b = (b << (4u - r)) | (b0 >> r);
  }
  if (LS > 1) {
    a <<= 4 * NB * sub;
    b <<= 4 * NB * sub;
  }
}

// Cut planes of this lane's sites of a half from its word's generator, whose
// state x comes before the value of the lane's highest site (masks_lcg_cut).
template <int LS>
__device__ __forceinline__ void lcg_half(uint32_t x, int sub, uint32_t cut_x, uint64_t cut_c,
                                         uint32_t& a, uint32_t& b) {
  constexpr int NB = 8 / LS;
  uint32_t acc[4] = {0, 0, 0, 0};
  uint32_t y = x + 0x80000000u;
  lcg_codes<NB>(acc, y, cut_x, cut_c);
  cut_planes(acc, a, b);
  if (LS > 1) {
    a <<= 4 * NB * sub;
    b <<= 4 * NB * sub;
  }
}

// The counts of `cnt` sweeps leave the LDS slots (one (anti, up) pair per
// wave and sweep): the first of them is sweep k0 of the launch (first sweep
// s0 of the lattice's series).
template <typename Lat>
__device__ __forceinline__ void drain_counts(const Lat& L, uint2* counts, int strip, int j,
                                             int64_t s0, int k0, int cnt) {
  for (int i = threadIdx.x; i < cnt; i += L.threads) {
    uint32_t anti = 0, up = 0;
    for (int w = 0; w < (L.threads >> 6); ++w) {
      anti += counts[i * kMaxWaves + w].x;
      up += counts[i * kMaxWaves + w].y;
      counts[i * kMaxWaves + w] = make_uint2(0, 0);
    }
    if (L.strips == 1) {
      const int64_t N = (int64_t)L.L * L.L;
      L.EM[2 * (s0 + k0 + i)] = 2 * (int64_t)anti - 2 * N;
      L.EM[2 * (s0 + k0 + i) + 1] = 2 * (int64_t)up - N;
    } else {
      uint32_t* p = L.part + 2 * (((size_t)(j & 1) * kBlockMaxK + k0 + i) * L.strips + strip);
      p[0] = anti;
      p[1] = up;
    }
  }
}

// (anti, up) added to a 64-bit LDS word, nothing returned, complete on return
// (a block barrier follows).  Written out: the compiler's atomic add first
// sums over the lanes, one readlane at a time.
__device__ __forceinline__ void lds_add(uint2* slot, uint32_t anti, uint32_t up) {
  const uint32_t addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint2*)slot;
  const uint64_t v = ((uint64_t)up << 32) | anti;
  asm volatile("ds_add_u64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : : "v"(addr), "v"(v) : "memory");
}

// x -> a x + b (mod 2^32): one or several steps of the generator at once.
struct Affine {
  uint32_t a, b;
};

__host__ __device__ inline Affine lcg_skip(uint64_t steps) {
  Affine r = {1u, 0u}, p = {kLcgA, kLcgC};
  for (; steps; steps >>= 1) {
    if (steps & 1) r = Affine{p.a * r.a, p.a * r.b + p.b};
    p = Affine{p.a * p.a, p.a * p.b + p.b};
  }
  return r;
}

// What the alternative dynamics keep beside the planes of a strip.
struct AltStrip {
  const uint32_t* lcg;   // LDS: the strip's generators as they were before the call
  Affine sweep;          // their advance to the current sweep (64 steps each)
  const uint32_t* pool;  // patterns (device memory)
  uint32_t shift, mask;
  uint32_t* starts;      // LDS: [2][kMaxGroups] start of every 256-word group, by step parity
  uint32_t first;        // global index of the strip's first word
  uint32_t group0;       // its group
  int groups;            // groups of the strip's words
  int wrapped;           // groups before the lattice's first word comes round again
};

// Starts of step s of the strip's groups for linear reads, by the first wave.
template <typename Lat>
__device__ __forceinline__ void pool_starts(const Lat& L, const AltStrip& x, int64_t s0, int s) {
  const int i = (int)threadIdx.x;
  if (i >= x.groups) return;
  uint32_t x0 = i < x.wrapped ? x.group0 + (uint32_t)i : (uint32_t)(i - x.wrapped);
  uint32_t x1 = 0, x2 = L.t + (uint32_t)(s0 + (s >> 1)), x3 = L.sid4 | (uint32_t)(s & 1);
  philox4x32_10(x0, x1, x2, x3, L.k0, L.k1);
  x.starts[(s & 1) * kMaxGroups + i] = x0 >> x.shift;
}

// K sweeps of the strip's R rows in LDS: local row r is global row y0 + r
// (mod L); rows H .. H + own - 1 are the strip's own.  A colour step's time
// is mostly a wave's chain of instructions, so lanes without work take the
// last row's and only their stores are left out (whole waves without work
// skip it), and with ONE (a single strip, one row per lane) everything but
// the uniforms and the spins is loop-invariant.
template <int LS, int MODE, bool ONE, bool SERIAL, typename Lat>
__device__ __forceinline__ void block_steps(const Lat& L, uint32_t* lds, uint2* counts, int strip,
                                            int j, int R, int H, int own, int y0, int64_t s0,
                                            int K, AltStrip alt) {
  constexpr int NB = 8 / LS;
  constexpr bool kAny = MODE == kAnyRow || MODE == kAnyRowCut;
  constexpr bool kPooled = MODE == kPool || MODE == kPoolLinear;
  constexpr bool kCutPlanes = MODE == kCut || MODE == kAnyRowCut || MODE == kLcg;
  // patterns come from memory: several rows' loads go out before the first is
  // used
  constexpr int kAhead = kPooled && !ONE ? 4 : 1;
  // few lanes count: they add in LDS; many: the wave sums first
  constexpr bool kAddCounts = LS >= 4;
  const bool wrap = ONE || L.strips == 1;
  const bool em = L.EM != nullptr, perturbed = L.perturb != 0;
  const int per = L.nh * LS, stride = 2 * L.W, pass = L.pass;
  int r0 = (int)threadIdx.x / per;
  const int hw = ((int)threadIdx.x - r0 * per) / LS, sub = (int)threadIdx.x % LS;
  const bool first_lane = sub == 0;
  if (r0 >= pass) r0 = 1 << 24;  // a lane of no row
  const bool last = hw == L.nh - 1;
  uint32_t mine = last && L.nbl < 32 ? (1u << L.nbl) - 1u : ~0u;  // valid sites of this lane
  const uint32_t valid = mine;
  if (LS > 1) mine &= ((1u << (4 * NB & 31)) - 1u) << (4 * NB * sub);
  // horizontal partners: bit 31 of the half to the left (the last valid bit
  // of the row for the first half), bit 0 of the half to the right
  const int hl = hw > 0 ? hw - 1 : L.nh - 1, hr = last ? 0 : hw + 1;
  const int shl = hw > 0 ? 31 : L.nbl - 1, shr = last ? L.nbl - 1 : 31;
  const uint32_t rowlen = kAny ? (uint32_t)L.half : (uint32_t)L.half >> 2;
  const uint32_t col = kAny ? 32u * hw + 4u * NB * sub : 8u * hw + NB * (uint32_t)sub;
  const uint32_t k0 = L.k0, k1 = L.k1, sid4 = L.sid4, t4 = L.t4, t8 = L.t8, cut_x = L.cut.x;
  const uint64_t cut_c = L.cut.c;
  const int side = L.L, wave = (int)threadIdx.x >> 6;
  const int plane = R * stride, lastrow = plane - stride;
  const int words = R * L.W;
  // the generator's values of this lane's sites follow this many others of
  // the word (site 63 takes the first)
  const Affine own_skip =
      MODE == kLcg ? lcg_skip((uint32_t)(64 - 32 * (hw & 1) - 4 * NB * (sub + 1))) : Affine{1u, 0u};
  const Affine sweep_skip = MODE == kLcg ? lcg_skip(64) : Affine{1u, 0u};
  // With two waves on a SIMD the loop is bound by instruction fetch as much as
  // by issue: its rare parts stand out of line (one taken branch per sweep),
  // and it is placed the same whatever code precedes it.  1000 sweeps of 64^2:
  // 0.89 ms; with the branches 0.90 to 1.01, by its place.
  asm volatile(".p2align 8");
  for (int k = 0; k < K; ++k) {
    const uint32_t t = L.t + (uint32_t)(s0 + k);
    uint2* const slot = &counts[(k & (kEmSlots - 1)) * kMaxWaves + wave];
    uint32_t anti = 0, up = 0;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int s = 2 * k + c;
      const int ra = wrap ? 0 : 1 + s, rb = wrap ? R - 1 : R - 2 - s;
      uint32_t* const self = lds + (c ? plane : 0);
      const uint32_t* const other = lds + (c ? 0 : plane);
      auto global_row = [&](int r) {
        const int y = y0 + r;
        return y >= side ? y - side : y;
      };
      // the two pattern halves of row `want` (or the last)
      auto pattern = [&](int want, uint32_t& a, uint32_t& b) {
        const int r = want < rb ? want : rb;
        const uint32_t iu = (uint32_t)(global_row(r) * L.W + (hw >> 1));
        uint32_t addr;
        if (MODE == kPoolLinear) {
          int g = (int)((iu >> 8) - alt.group0);
          if (iu < alt.first) g = (int)(iu >> 8) + alt.wrapped;
          addr = (alt.starts[c * kMaxGroups + g] + (iu & 255u)) & alt.mask;
        } else {
          uint32_t x0 = iu, x1 = 0, x2 = t, x3 = sid4 | (uint32_t)c;
          philox4x32_10(x0, x1, x2, x3, k0, k1);
          addr = x0 >> alt.shift;
        }
        const uint32_t* p = alt.pool + 4 * (size_t)addr + (hw & 1);
        a = p[0];
        b = p[2];
      };
      // one row of the step; pools: (a, b) are given
      auto row = [&](int want, uint32_t a, uint32_t b) {
        const int r = want < rb ? want : rb;
        const int y = global_row(r);
        const int at = (int)__umul24((uint32_t)r, (uint32_t)stride);
        const int am = wrap && r == 0 ? lastrow : at - stride;
        const int ap = wrap && at == lastrow ? 0 : at + stride;
        const uint32_t left = (uint32_t)(((y + c) & 1) - 1);  // all ones: the partner is left
        const uint32_t s_old = self[at + hw], n0 = other[at + hw];
        const uint32_t n2 = other[am + hw], n3 = other[ap + hw];
        const uint32_t sd = other[at + (left ? hl : hr)];
        if (MODE == kLcg) {
          uint32_t x = alt.lcg[(c ? words : 0) + (at >> 1) + (hw >> 1)];
          x = alt.sweep.a * x + alt.sweep.b;
          lcg_half<LS>(own_skip.a * x + own_skip.b, sub, cut_x, cut_c, a, b);
        } else if (!kPooled) {
          half_planes<LS, MODE, SERIAL>((uint32_t)y * rowlen + col, sub, k0, k1, t,
                                        sid4 | (uint32_t)c, t4, t8, cut_x, cut_c, a, b);
        }
        const uint32_t n1 = bfi(left, (n0 << 1) | (sd >> shl), (n0 >> 1) | (sd << shr));
        uint32_t f = kCutPlanes ? flip_half_cut(s_old, n0, n1, n2, n3, a, b)
                                : flip_half(s_old, n0, n1, n2, n3, a, b);
        f = lanes_or<LS>(f & mine);
        const uint32_t s_new = s_old ^ f;
        const bool store = first_lane && want <= rb;
        if (store) self[at + hw] = s_new;
        if (c == 1 && em) {
          const bool on = store && (uint32_t)(r - H) < (uint32_t)own;
          const uint32_t da = __popc(s_new ^ n0) + __popc((s_new ^ n1) & valid) +
                              __popc(s_new ^ n2) + __popc(s_new ^ n3);
          const uint32_t du = __popc(s_new) + __popc(n0);
          anti += on ? da : 0u;
          up += on ? du : 0u;
        }
      };
      if (ONE) {
        uint32_t a = 0, b = 0;
        if (kPooled) pattern(r0, a, b);
        row(r0, a, b);
      } else {
        for (int base = ra; base <= rb; base += pass * kAhead) {
          uint32_t a[kAhead], b[kAhead];
          // the wave's first lane has its smallest row
          if (__builtin_amdgcn_readfirstlane(base + r0) > rb) continue;
          if (kPooled) {
#pragma unroll
            for (int i = 0; i < kAhead; ++i) pattern(base + r0 + i * pass, a[i], b[i]);
          }
#pragma unroll
          for (int i = 0; i < kAhead; ++i)
            if (i == 0 || __builtin_amdgcn_readfirstlane(base + r0 + i * pass) <= rb)
              row(base + r0 + i * pass, a[i], b[i]);
        }
      }
      if (c == 1 && em) {
        if (kAddCounts) {
          if (first_lane) lds_add(slot, anti, up);
        } else {
          const uint32_t wa = wave_total(anti), wu = wave_total(up);
          if ((threadIdx.x & 63) == 63) *slot = make_uint2(wa, wu);
        }
      }
      if (MODE == kPoolLinear) pool_starts(L, alt, s0, s + 1);
      if (__builtin_expect(perturbed, 0)) perturb_wave(L.perturb, (uint32_t)s);
      __syncthreads();
    }
    if (MODE == kLcg)
      alt.sweep = Affine{sweep_skip.a * alt.sweep.a, sweep_skip.a * alt.sweep.b + sweep_skip.b};
    // the slots are written again only after the next colour-0 barrier
    if (__builtin_expect(em && ((k & (kEmSlots - 1)) == kEmSlots - 1 || k == K - 1), 0))
      drain_counts(L, counts, strip, j, s0, k & ~(kEmSlots - 1), (k & (kEmSlots - 1)) + 1);
  }
}

// The same for the pools with a whole word per lane: the VALU bounds a step
// (75 instructions a half, of which the flip takes 18), and a word's address,
// row and neighbours cost what a half's do.  us per sweep of a linear pool with
// a half and a word per lane: 2048^2 3.5, 2.65; 8192^2 7.8, 5.6; 16384^2 22.4,
// 16.1; random addresses are bound by memory either way.
template <int MODE, typename Lat>
__device__ __forceinline__ void pool_word_steps(const Lat& L, uint64_t* lds, uint2* counts,
                                                int strip, int j, int R, int H, int own, int y0,
                                                int64_t s0, int K, const AltStrip& alt) {
  constexpr int kAhead = 4;  // rows whose patterns are on their way
  const bool wrap = L.strips == 1, em = L.EM != nullptr, perturbed = L.perturb != 0;
  const int W = L.W, pass = L.pass, side = L.L, wave = (int)threadIdx.x >> 6;
  int r0 = (int)threadIdx.x / W;
  const int w = (int)threadIdx.x - r0 * W;
  if (r0 >= pass) r0 = 1 << 24;  // a lane of no row
  const bool last = w == W - 1;
  const int nb = L.half - 64 * (W - 1);  // sites of a row's last word
  const uint64_t valid = last && nb < 64 ? (1ull << nb) - 1ull : ~0ull;
  const int wl = w > 0 ? w - 1 : W - 1, wr = last ? 0 : w + 1;
  const int shl = w > 0 ? 63 : nb - 1, shr = last ? nb - 1 : 63;
  const int plane = R * W, lastrow = plane - W;
  const ulonglong2* const pool = (const ulonglong2*)alt.pool;
  asm volatile(".p2align 8");
  for (int k = 0; k < K; ++k) {
    uint2* const slot = &counts[(k & (kEmSlots - 1)) * kMaxWaves + wave];
    uint32_t anti = 0, up = 0;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int s = 2 * k + c;
      const int ra = wrap ? 0 : 1 + s, rb = wrap ? R - 1 : R - 2 - s;
      uint64_t* const self = lds + (c ? plane : 0);
      const uint64_t* const other = lds + (c ? 0 : plane);
      auto global_row = [&](int r) {
        const int y = y0 + r;
        return y >= side ? y - side : y;
      };
      auto pattern = [&](int want) {
        const uint32_t iu = (uint32_t)(global_row(want < rb ? want : rb) * W + w);
        uint32_t addr;
        if (MODE == kPoolLinear) {
          int g = (int)((iu >> 8) - alt.group0);
          if (iu < alt.first) g = (int)(iu >> 8) + alt.wrapped;
          addr = (alt.starts[c * kMaxGroups + g] + (iu & 255u)) & alt.mask;
        } else {
          uint32_t x0 = iu, x1 = 0, x2 = L.t + (uint32_t)(s0 + k), x3 = L.sid4 | (uint32_t)c;
          philox4x32_10(x0, x1, x2, x3, L.k0, L.k1);
          addr = x0 >> alt.shift;
        }
        return pool[addr];
      };
      auto row = [&](int want, ulonglong2 ab) {
        const int r = want < rb ? want : rb;
        const int at = (int)__umul24((uint32_t)r, (uint32_t)W);
        const int am = wrap && r == 0 ? lastrow : at - W;
        const int ap = wrap && at == lastrow ? 0 : at + W;
        const bool left = ((global_row(r) + c) & 1) == 0;
        const uint64_t s_old = self[at + w], n0 = other[at + w];
        const uint64_t n2 = other[am + w], n3 = other[ap + w];
        const uint64_t sd = other[at + (left ? wl : wr)];
        const uint64_t n1 = left ? (n0 << 1) | (sd >> shl) : (n0 >> 1) | (sd << shr);
        const uint32_t lo = flip_half((uint32_t)s_old, (uint32_t)n0, (uint32_t)n1, (uint32_t)n2,
                                      (uint32_t)n3, (uint32_t)ab.x, (uint32_t)ab.y);
        const uint32_t hi = flip_half((uint32_t)(s_old >> 32), (uint32_t)(n0 >> 32),
                                      (uint32_t)(n1 >> 32), (uint32_t)(n2 >> 32),
                                      (uint32_t)(n3 >> 32), (uint32_t)(ab.x >> 32),
                                      (uint32_t)(ab.y >> 32));
        const uint64_t s_new = s_old ^ ((((uint64_t)hi << 32) | lo) & valid);
        const bool store = want <= rb;
        if (store) self[at + w] = s_new;
        if (c == 1 && em) {
          const bool on = store && (uint32_t)(r - H) < (uint32_t)own;
          const uint32_t da = __popcll(s_new ^ n0) + __popcll((s_new ^ n1) & valid) +
                              __popcll(s_new ^ n2) + __popcll(s_new ^ n3);
          const uint32_t du = __popcll(s_new) + __popcll(n0);
          anti += on ? da : 0u;
          up += on ? du : 0u;
        }
      };
      for (int base = ra; base <= rb; base += pass * kAhead) {
        ulonglong2 ab[kAhead];
        // the wave's first lane has its smallest row
        if (__builtin_amdgcn_readfirstlane(base + r0) > rb) continue;
#pragma unroll
        for (int i = 0; i < kAhead; ++i) ab[i] = pattern(base + r0 + i * pass);
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
          if (i == 0 || __builtin_amdgcn_readfirstlane(base + r0 + i * pass) <= rb)
            row(base + r0 + i * pass, ab[i]);
      }
      if (c == 1 && em) {
        const uint32_t wa = wave_total(anti), wu = wave_total(up);
        if ((threadIdx.x & 63) == 63) *slot = make_uint2(wa, wu);
      }
      if (MODE == kPoolLinear) pool_starts(L, alt, s0, s + 1);
      if (__builtin_expect(perturbed, 0)) perturb_wave(L.perturb, (uint32_t)s);
      __syncthreads();
    }
    if (__builtin_expect(em && ((k & (kEmSlots - 1)) == kEmSlots - 1 || k == K - 1), 0))
      drain_counts(L, counts, strip, j, s0, k & ~(kEmSlots - 1), (k & (kEmSlots - 1)) + 1);
  }
}

// One wave's share of the partials of one sweep (kBlockMaxStrips / 64 strips
// per lane).
struct Parts {
  uint2 v[kBlockMaxStrips / 64];
};

// Loads the partials of sweep k of launch j (kept apart from their sum, so
// that the loads can be issued long before it).
template <typename Lat>
__device__ __forceinline__ Parts load_parts(const Lat& L, int j, int k) {
  const uint2* p = (const uint2*)L.part + ((size_t)(j & 1) * kBlockMaxK + k) * L.strips;
  Parts q;
#pragma unroll
  for (int i = 0; i < kBlockMaxStrips / 64; ++i) {
    const int at = (int)(threadIdx.x & 63) + 64 * i;
    q.v[i] = at < L.strips ? p[at] : make_uint2(0, 0);
  }
  return q;
}

// (E, M) of sweep s of the lattice's series (sums below 2^32: L <= kBlockMaxL).
template <typename Lat>
__device__ __forceinline__ void store_parts(const Lat& L, const Parts& q, int64_t s) {
  uint32_t anti = 0, up = 0;
#pragma unroll
  for (int i = 0; i < kBlockMaxStrips / 64; ++i) {
    anti += q.v[i].x;
    up += q.v[i].y;
  }
  anti = wave_total(anti);
  up = wave_total(up);
  if ((threadIdx.x & 63) == 63) {
    const int64_t N = (int64_t)L.L * L.L;
    L.EM[2 * s] = 2 * (int64_t)anti - 2 * N;
    L.EM[2 * s + 1] = 2 * (int64_t)up - N;
  }
}

// The sweeps first, first + step, ... of the last launch, by one wave.
template <typename Lat>
__device__ __forceinline__ void reduce_last(const Lat& L, int first, int step) {
  const int j = L.launches - 1;
  const int64_t s0 = sweeps_before(L.n, j, L.launches);
  for (int k = first; s0 + k < L.n; k += step) store_parts(L, load_parts(L, j, k), s0 + k);
}

// Lat: BlockLattice, as a kernel argument or in a table (constant memory).
// ALT: the alternative dynamics x of a lone lattice instead of Philox.
template <bool ALT, bool SERIAL, typename Lat>
__device__ __forceinline__ void block_run(const Lat& L, const BlockAlt* x, int strip, int j,
                                          uint32_t* lds) {
  __shared__ uint2 counts[kEmSlots * kMaxWaves];
  __shared__ uint32_t starts[ALT ? 2 * kMaxGroups : 1];
  // what the plans leave for them (an unused array takes none)
  static_assert(sizeof(counts) + (ALT ? sizeof(starts) : 0) ==
                    (size_t)block_static_lds(ALT ? kBlockLcg : kBlockPhilox),
                "block_static_lds");
  // waves beyond this lattice's share of the workgroup leave at once
  if ((int)(threadIdx.x & ~63u) >= L.threads || j >= L.launches) return;
  const bool wrap = L.strips == 1;
  const int64_t s0 = sweeps_before(L.n, j, L.launches);
  const int K = (int)(sweeps_before(L.n, j + 1, L.launches) - s0);
  const int H = wrap ? 0 : 2 * K;
  const int row0 = strip * L.rows;
  const int own = L.L - row0 < L.rows ? L.L - row0 : L.rows;
  const int R = own + 2 * H;
  int y0 = row0 - H;
  y0 = y0 < 0 ? y0 + L.L : y0;
  const int W = L.W, all = L.L * W;
  const uint64_t* src = L.buf[wrap ? 0 : (j & 1)];
  uint64_t* dst = L.buf[wrap ? 0 : ((j + 1) & 1)];
  uint64_t* lds64 = (uint64_t*)lds;
  for (int i = threadIdx.x; i < kEmSlots * kMaxWaves; i += L.threads) counts[i] = make_uint2(0, 0);
  for (int i = threadIdx.x; i < R * W; i += L.threads) {
    int p = y0 * W + i;
    p = p >= all ? p - all : p;
    lds64[i] = src[p];
    lds64[R * W + i] = src[all + p];
    if (ALT && x->kind == kBlockLcg) {
      lds[4 * R * W + i] = x->lcg[p];
      lds[5 * R * W + i] = x->lcg[all + p];
    }
  }
  AltStrip alt = {};
  if (ALT) {
    alt.lcg = lds + 4 * R * W;
    alt.sweep = lcg_skip(64 * (uint64_t)s0);
    alt.pool = (const uint32_t*)x->pool;
    alt.shift = x->pool_shift;
    alt.mask = x->pool_mask;
    alt.starts = starts;
    alt.first = (uint32_t)(y0 * W);
    alt.group0 = alt.first >> 8;
    const int end = y0 * W + R * W;  // past `all` when the strip's rows wrap
    alt.wrapped = (((end < all ? end : all) - 1) >> 8) - (int)alt.group0 + 1;
    alt.groups = alt.wrapped + (end > all ? ((end - all - 1) >> 8) + 1 : 0);
    if (x->kind == kBlockPoolLinear) pool_starts(L, alt, s0, 0);
  }
  // the first strips reduce the E/M partials of the launch before, one sweep
  // each (a launch has fewer sweeps than strips); loaded now, summed at the end
  const int64_t sp = wrap || j == 0 ? s0 : sweeps_before(L.n, j - 1, L.launches);
  const bool reduce = L.EM != nullptr && sp + strip < s0 && threadIdx.x < 64;
  Parts parts;
  if (reduce) parts = load_parts(L, j - 1, strip);
  __syncthreads();
#define ISING_BLOCK(LS, MODE)                                                           \
  do {                                                                                  \
    if (wrap && R <= L.pass)                                                            \
      block_steps<LS, MODE, true, SERIAL>(L, lds, counts, strip, j, R, H, own, y0, s0,  \
                                          K, alt);                                      \
    else                                                                                \
      block_steps<LS, MODE, false, SERIAL>(L, lds, counts, strip, j, R, H, own, y0, s0, \
                                           K, alt);                                     \
  } while (0)
  if constexpr (ALT) {
    if (L.ls == 0 && x->kind == kBlockPool) {
      pool_word_steps<kPool>(L, lds64, counts, strip, j, R, H, own, y0, s0, K, alt);
    } else if (L.ls == 0) {
      pool_word_steps<kPoolLinear>(L, lds64, counts, strip, j, R, H, own, y0, s0, K, alt);
    } else if (x->kind == kBlockPool) {
      ISING_BLOCK(1, kPool);
    } else if (x->kind == kBlockPoolLinear) {
      ISING_BLOCK(1, kPoolLinear);
    } else {
      switch (L.ls) {
        case 8: ISING_BLOCK(8, kLcg); break;
        case 4: ISING_BLOCK(4, kLcg); break;
        case 2: ISING_BLOCK(2, kLcg); break;
        default: ISING_BLOCK(1, kLcg); break;
      }
    }
  } else if ((L.half & 3) != 0) {
    if (L.ls == 8)
      ISING_BLOCK(8, kAnyRow);
    else if (L.ls == 4)
      ISING_BLOCK(4, kAnyRow);
    else if (L.cut.x != 0 && L.ls == 2)
      ISING_BLOCK(2, kAnyRowCut);
    else if (L.cut.x != 0)
      ISING_BLOCK(1, kAnyRowCut);
    else if (L.ls == 2)
      ISING_BLOCK(2, kAnyRow);
    else
      ISING_BLOCK(1, kAnyRow);
  } else if (L.ls >= 4) {
    // one or two blocks per lane: the transpose of the cut costs as much as
    // the compares it saves
    if (L.ls == 8)
      ISING_BLOCK(8, kCompare);
    else
      ISING_BLOCK(4, kCompare);
  } else if (L.cut.x != 0) {
    if (L.ls == 2)
      ISING_BLOCK(2, kCut);
    else
      ISING_BLOCK(1, kCut);
  } else {
    if (L.ls == 2)
      ISING_BLOCK(2, kCompare);
    else
      ISING_BLOCK(1, kCompare);
  }
#undef ISING_BLOCK
  for (int i = threadIdx.x; i < own * W; i += L.threads) {
    __hip_atomic_store(&dst[row0 * W + i], lds64[H * W + i], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&dst[all + row0 * W + i], lds64[(R + H) * W + i], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
  if (reduce) store_parts(L, parts, sp + strip);
}

__global__ __launch_bounds__(1024) void k_block(BlockLattice L, int j) {
  extern __shared__ uint64_t block_lds[];
  block_run<false, false>(L, nullptr, blockIdx.x, j, (uint32_t*)block_lds);
}

// The paper's generators and pools.
__global__ __launch_bounds__(1024) void k_block_alt(BlockLattice L, BlockAlt x, int j) {
  extern __shared__ uint64_t block_lds[];
  block_run<true, false>(L, &x, blockIdx.x, j, (uint32_t*)block_lds);
}

// All generators `skip` steps on (the strips of a call derive their states
// from those before it, so the caller's buffer changes once).
__global__ __launch_bounds__(256) void k_lcg_advance(uint32_t* state, int64_t n, Affine skip) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    state[i] = skip.a * state[i] + skip.b;
}

// The same for a table of lattices; tasks are (lattice, strip).  Up to one
// task per compute unit, a task has its SIMDs to itself and its blocks
// interleave (SERIAL: no, 113 VGPRs); more tasks share them, two workgroups of
// 16 waves at a time (63 VGPRs).  1000 sweeps of 24 lattices of 8^2 to 64^2:
// 1.15 ms against 1.20 with SERIAL (0.15 of both on the host); a queue of 24
// requests up to 2048^2: 27.0 ms all interleaved, 25.8 all SERIAL, 25.4 by this
// rule.
template <bool SERIAL>
__device__ __forceinline__ void block_many(const BlockLattice* tab, const BlockTask* tasks,
                                           int j) {
  extern __shared__ uint64_t block_lds[];
  const BlockTask task = ((const BlockTask ISING_CONSTANT_AS*)tasks)[blockIdx.x];
  block_run<false, SERIAL>(((const BlockLattice ISING_CONSTANT_AS*)tab)[task.lattice], nullptr,
                           task.strip, j, (uint32_t*)block_lds);
}

__global__ __launch_bounds__(1024) void k_block_few(const BlockLattice* tab,
                                                    const BlockTask* tasks, int j) {
  block_many<false>(tab, tasks, j);
}

__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) void k_block_many(
    const BlockLattice* tab, const BlockTask* tasks, int j) {
  block_many<true>(tab, tasks, j);
}

// (E, M) of every lattice's last launch.
__global__ __launch_bounds__(64) void k_block_finalize(BlockLattice L) {
  reduce_last(L, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(64) void k_block_finalize_many(const BlockLattice* tab) {
  const auto& L = ((const BlockLattice ISING_CONSTANT_AS*)tab)[blockIdx.x];
  if (L.EM != nullptr && L.strips > 1) reduce_last(L, 0, 1);
}

}  // namespace

// ---------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------

BlockLattice block_lattice(const ising_lattice* h, const BlockShape& s, int64_t n,
                           bool one_launch, int64_t* EM) {
  BlockLattice b;
  std::memset(&b, 0, sizeof(b));
  b.buf[0] = h->planes;
  b.buf[1] = h->spare;
  b.L = (int32_t)h->L;
  b.W = h->g.W;
  b.half = (int32_t)h->g.half;
  b.nh = (b.half + 31) / 32;
  b.nbl = b.half - 32 * (b.nh - 1);
  b.rows = s.rows;
  b.strips = s.strips;
  b.ls = s.ls;
  b.pass = s.pass;
  b.threads = s.threads;
  b.launches = (int32_t)block_launches(s, n, one_launch);
  b.k0 = (uint32_t)h->seed;
  b.k1 = (uint32_t)(h->seed >> 32);
  b.sid4 = h->stream_id << 2;
  b.t = (uint32_t)h->sweep;
  b.t4 = h->t4;
  b.t8 = h->t8;
  b.cut = h->cut;
  b.n = n;
  b.EM = EM;
  b.part = (uint32_t*)h->part[0];
  b.perturb = debug_perturb_seed();
  return b;
}

// Dynamics of a handle as the block kernels know them, or -1 where they have
// none (generators without a cut of their thresholds).
int block_kind(const ising_lattice* h) {
  if (h->pool) return h->pool_linear ? kBlockPoolLinear : kBlockPool;
  if (h->lcg) return h->lcut.x ? kBlockLcg : -1;
  return kBlockPhilox;
}

ising_status enqueue_block_sweeps(ising_lattice* h, const BlockShape& s, int64_t n,
                                  int64_t* dev_EM) {
  BlockLattice b = block_lattice(h, s, n, true, dev_EM);
  BlockAlt x = {};
  x.kind = block_kind(h);
  if (x.kind == kBlockLcg) {
    b.cut = h->lcut;
    x.lcg = h->lcg;
  } else if (x.kind != kBlockPhilox) {
    x.pool = h->pool;
    x.pool_shift = (uint32_t)(32 - h->pool_m);
    x.pool_mask = (uint32_t)((1ull << h->pool_m) - 1);
  }
  for (int32_t j = 0; j < b.launches; ++j) {
    if (x.kind == kBlockPhilox)
      hipLaunchKernelGGL(k_block, dim3(s.strips), dim3(s.threads), s.lds, h->stream, b, j);
    else
      hipLaunchKernelGGL(k_block_alt, dim3(s.strips), dim3(s.threads), s.lds, h->stream, b, x, j);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "block sweep launch");
  }
  if (s.strips > 1 && dev_EM) {
    hipLaunchKernelGGL(k_block_finalize, dim3(s.sweeps), dim3(64), 0, h->stream, b);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "block E/M finalisation launch");
  }
  if (x.kind == kBlockLcg) {
    const int64_t words = 2 * h->plane_words;
    hipLaunchKernelGGL(k_lcg_advance, dim3((unsigned)std::min<int64_t>((words + 255) / 256, 2048)),
                       dim3(256), 0, h->stream, h->lcg, words, lcg_skip(64 * (uint64_t)n));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "generator advance launch");
  }
  return ISING_OK;
}

hipError_t launch_block_many(hipStream_t st, const BlockLattice* tab, const BlockTask* tasks,
                             int ntasks, int cus, int threads, size_t lds, int j) {
  if (ntasks <= cus)
    hipLaunchKernelGGL(k_block_few, dim3(ntasks), dim3(threads), lds, st, tab, tasks, j);
  else
    hipLaunchKernelGGL(k_block_many, dim3(ntasks), dim3(threads), lds, st, tab, tasks, j);
  return hipGetLastError();
}

hipError_t launch_block_finalize_many(hipStream_t st, const BlockLattice* tab, int nlat) {
  hipLaunchKernelGGL(k_block_finalize_many, dim3(nlat), dim3(64), 0, st, tab);
  return hipGetLastError();
}

}  // namespace ising
