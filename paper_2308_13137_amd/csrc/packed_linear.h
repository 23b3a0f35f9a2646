// The packed linear Y = X W^T + B over Eq. 2's codes (W = (q - z) h per group):
// its kernels and launch rules, one code width at a time; each
// packed_linear_bNN.hip instantiates two widths (they compile in parallel).
//
//   packed_mfma_kernel    up to 96 tokens, in launches of at most 32: matrix
//                         cores fed by asynchronous copies, bound by the stream
//                         of codes at few tokens
//   packed_wide_kernel    25 to 32 of them where rows are many or codes wide
//   packed_tile_kernel    more tokens: a tiled product
//   packed_linear_kernel  one or two tokens with groups that are no multiple of 128
//
// No kernel rounds a weight: codes enter the products as exact small integers in
// bf16, and step sizes and zero points multiply fp32 sums.  Measured over a 7B
// block's four stacked linears (W g128, 4 blocks, one graph; against the vector
// kernel at up to 7 tokens and the former matrix-core kernel above):
//   W4, 1 token 38.4 -> 37.1 us; W3, 1 token 44.9 -> 38.1; W4, 4 tokens 66 -> 43;
//   8 tokens 51 -> 45; 16 tokens 57 -> 49; W3, 24 tokens 80 -> 63; W2 g64 (13B),
//   4 tokens 103 -> 66; W4, 500 tokens 1274 -> 450.
// Against 64-bit sums the results are 4 to 40 times closer than before (the codes'
// offset is 2^BITS instead of 128, so less cancels).
#pragma once
#include <algorithm>
#include <mutex>
#include <vector>

#include "common.h"
#include "packed.h"

namespace oq {
namespace {

constexpr size_t PL_LDS_MAX = 160 * 1024;
constexpr int PL_THREADS = 256;               // vector kernel: 4 waves
constexpr int PL_WAVES = PL_THREADS / 64;
constexpr int PL_ROWS = 2;                    // output rows a wave works on together
constexpr int PL_U = 2;                       // runs per lane loaded together
constexpr uint32_t BF16_128_PAIR = 0x43004300u;

// ------------------------------------------------------------------ codes to bf16
// A run's 32 codes are consumed as 16 pairs (p, p + 16): the run's bit string
// is two streams of 16 codes, `BITS` 16-bit half-words each, and interleaving
// them half-word by half-word (one v_perm each) puts both codes of a pair at
// the same offset of the two halves of a dword.
//
// A code is widened without a conversion: shifted to the top of the mantissa
// field and OR-ed into the bf16 value 2^BITS it gives exactly 2^BITS + q.
typedef __bf16 bf16x2_v __attribute__((ext_vector_type(2)));

// A constant the compiler does not see as one: (a & m) | c is then a single
// v_and_or_b32 (with literal operands, which a gfx9 three-operand instruction
// does not take, it would be an AND and an OR).
OQ_DEV uint32_t opaque_s(uint32_t v) {
  uint32_t r;
  asm("s_mov_b32 %0, %1" : "=s"(r) : "i"(v));
  return r;
}
OQ_DEV uint32_t opaque_v(uint32_t v) {
  uint32_t r;
  asm("v_mov_b32 %0, %1" : "=v"(r) : "i"(v));
  return r;
}

// Masks of a pair's bits: the whole code, and for a code that spans two
// half-words with n1 = 1 .. BITS - 1 bits in the first, both pieces.
template <int BITS>
struct CodeMasks {
  uint32_t magic, whole, lo[BITS], hi[BITS];
  OQ_DEV CodeMasks() {
    constexpr int T = 7 - BITS;
    magic = opaque_v(uint32_t((127 + BITS) << 7) * 0x10001u);
    whole = opaque_s((((1u << BITS) - 1) << T) * 0x10001u);
#pragma unroll
    for (int n1 = 1; n1 < BITS; ++n1) {
      lo[n1] = opaque_s((((1u << n1) - 1) << T) * 0x10001u);
      hi[n1] = opaque_s((((1u << (BITS - n1)) - 1) << (T + n1)) * 0x10001u);
    }
  }
};

template <int BITS>
OQ_DEV void interleave_run(const uint32_t (&w)[BITS], uint32_t (&R)[BITS]) {
#pragma unroll
  for (int k = 0; k < BITS; ++k) {
    const int hk = k + BITS;
    R[k] = __builtin_amdgcn_perm(w[hk >> 1], w[k >> 1],
                                 ((hk & 1) ? 0x07060000u : 0x05040000u) | ((k & 1) ? 0x0302u : 0x0100u));
  }
}

// v << n (n > 0) or v >> -n
OQ_DEV uint32_t shift_by(uint32_t v, int n) { return n >= 0 ? v << n : v >> -n; }

// The pair (2^BITS + q_p, 2^BITS + q_{p + 16}) of an interleaved run as two bf16.
template <int BITS>
OQ_DEV uint32_t code_pair(const uint32_t (&R)[BITS], int p, const CodeMasks<BITS>& cm) {
  constexpr int T = 7 - BITS;
  const int k = (BITS * p) >> 4, s = (BITS * p) & 15;
  if (s + BITS <= 16) return (shift_by(R[k], T - s) & cm.whole) | cm.magic;
  const int n1 = 16 - s;                                  // bits in half-word k
  const uint32_t v = (shift_by(R[k], T - s) & cm.lo[n1]) | cm.magic;
  return (shift_by(R[k + 1], T + n1) & cm.hi[n1]) | v;
}

// codes 4 m .. 4 m + 3 and 16 + 4 m .. of a run as a matrix operand (m 0..3)
template <int BITS>
OQ_DEV bf16x8_t code_frag(const uint32_t (&R)[BITS], int m, const CodeMasks<BITS>& cm) {
  return __builtin_bit_cast(bf16x8_t, make_uint4(code_pair<BITS>(R, 4 * m, cm),
                                                 code_pair<BITS>(R, 4 * m + 1, cm),
                                                 code_pair<BITS>(R, 4 * m + 2, cm),
                                                 code_pair<BITS>(R, 4 * m + 3, cm)));
}

OQ_DEV float dot2_bf16(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_v, a),
                                         __builtin_bit_cast(bf16x2_v, b), c, false);
}

// one run: BITS dwords, 4-byte aligned (16 for 4 bits, 8 for 2)
template <int BITS>
OQ_DEV void load_run(const uint32_t* __restrict__ src, uint32_t (&w)[BITS]) {
  if constexpr (BITS == 4) {
    const uint4 v = *reinterpret_cast<const uint4*>(src);
    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
  } else if constexpr (BITS == 2) {
    const uint2 v = *reinterpret_cast<const uint2*>(src);
    w[0] = v.x; w[1] = v.y;
  } else {
#pragma unroll
    for (int k = 0; k < BITS; ++k) w[k] = src[k];
  }
}

// Buffer loads of N dwords at byte offset `off`: past the descriptor's size they
// read zeros and touch no memory, so a pipelined loop can issue them without a
// branch (a branch around loads makes the compiler wait for all of them where
// the paths meet).
typedef __amdgpu_buffer_rsrc_t rsrc_t;
OQ_DEV rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00027000);
}
template <int N>
OQ_DEV void buffer_load(rsrc_t r, uint32_t off, uint32_t* v) {
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  typedef uint32_t u3 __attribute__((ext_vector_type(3)));
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  if constexpr (N == 1) {
    v[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
  } else if constexpr (N == 2) {
    const u2 q = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
    v[0] = q.x; v[1] = q.y;
  } else if constexpr (N == 3) {
    const u3 q = __builtin_amdgcn_raw_buffer_load_b96(r, off, 0, 0);
    v[0] = q.x; v[1] = q.y; v[2] = q.z;
  } else {
    const u4 q = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    if constexpr (N > 4) buffer_load<N - 4>(r, off + 16, v + 4);
  }
}

// Eight channels of a token's lower and of its upper half run, interleaved
// into the pair order: u0 the first four pairs, u1 the last four.
OQ_DEV void interleave_x(uint4 lo, uint4 hi, uint4& u0, uint4& u1) {
  constexpr uint32_t EV = 0x05040100u, OD = 0x07060302u;
  u0 = make_uint4(__builtin_amdgcn_perm(hi.x, lo.x, EV), __builtin_amdgcn_perm(hi.x, lo.x, OD),
                  __builtin_amdgcn_perm(hi.y, lo.y, EV), __builtin_amdgcn_perm(hi.y, lo.y, OD));
  u1 = make_uint4(__builtin_amdgcn_perm(hi.z, lo.z, EV), __builtin_amdgcn_perm(hi.z, lo.z, OD),
                  __builtin_amdgcn_perm(hi.w, lo.w, EV), __builtin_amdgcn_perm(hi.w, lo.w, OD));
}

// wave-private LDS written by some lanes and read by others: the hardware
// keeps a wave's LDS accesses in order, this keeps the compiler from moving
// them across it
OQ_DEV void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Workgroup barrier that waits for LDS traffic only: global loads issued
// before it (the next tiles' codes) stay in flight across it.
OQ_DEV void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The group of a 32-channel part: part / (group / 32) as a multiplication by
// group_inv = ceil(2^31 / (group / 32)), exact for parts and groups of up to
// PACKED_MAX_C_IN / 32 = 2048 (2048 * 2048 < 2^31).
OQ_DEV int group_of(int part, uint32_t group_inv) { return int(__umulhi(uint32_t(part) << 1, group_inv)); }

// ------------------------------------------------------------------ pair order
// A run's 32 codes are consumed as 16 pairs.  For 4- and 2-bit codes a pair is
// two fields 16 bits apart in one dword, so one AND/OR extracts both; other
// widths pair neighbours.  The activation row is staged in LDS in the same
// pair order: pair p multiplies activations pair_lo(p) (low half) and
// pair_hi(p) (high half) of the run.
template <int BITS>
OQ_DEV constexpr int pair_lo(int p) {
  return BITS == 4 ? 8 * (p >> 2) + (p & 3) : BITS == 2 ? 16 * (p >> 3) + (p & 7) : 2 * p;
}
template <int BITS>
OQ_DEV constexpr int pair_hi(int p) {
  return BITS == 4 ? pair_lo<BITS>(p) + 4 : BITS == 2 ? pair_lo<BITS>(p) + 8 : 2 * p + 1;
}

// bits pos .. pos + BITS - 1 of the run's string (pos known at compile time)
template <int BITS>
OQ_DEV uint32_t field(const uint32_t* w, int pos) {
  const int d = pos >> 5, o = pos & 31;
  uint32_t v = w[d] >> o;
  if (o + BITS > 32) v |= w[d + 1] << (32 - o);
  return v & ((1u << BITS) - 1);
}

// (a & mask) | magic in one instruction.  The compiler emits an AND and an OR
// here: both constants are literals, and a gfx9 three-operand instruction
// takes no literal, so they are passed in registers.
OQ_DEV uint32_t and_or(uint32_t a, uint32_t mask, uint32_t magic) {
  uint32_t r;
  asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(mask), "v"(magic));
  return r;
}

// The 16 pairs of bf16 values (128 + q_lo, 128 + q_hi) of one run.
template <int BITS>
OQ_DEV void code_pairs(const uint32_t* w, uint32_t* p, uint32_t mask, uint32_t magic) {
  if constexpr (BITS == 4) {
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
      for (int i = 0; i < 4; ++i) p[4 * d + i] = and_or(w[d] >> (4 * i), mask, magic);
  } else if constexpr (BITS == 2) {
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int i = 0; i < 8; ++i) p[8 * d + i] = and_or(w[d] >> (2 * i), mask, magic);
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      p[i] = field<BITS>(w, 2 * i * BITS) | (field<BITS>(w, (2 * i + 1) * BITS) << 16) | BF16_128_PAIR;
  }
}

// ------------------------------------------------------------------ one or two tokens, small groups
// Groups that are no multiple of 128 (32, 64, 96, ..) at one or two tokens: a product per part would
// leave the matrix cores mostly zeros, so the dot-product unit takes the runs
// one by one (4096 channels, W4, one token, groups of 32: 43.9 us over a 7B
// block's linears, 61.6 us on matrix cores; groups of 64: 35.7 against 48.5 us
// at W2; from three tokens the matrix cores are faster, 64.1 -> 53.1 us).  With
// p = sum x (128 + q) over a 32-code run and xs = sum x over the same run, that
// run contributes h (p - (128 + z) xs).
//
// LDS: for token t and run k, the 16 activation pairs as four 16-byte quads at
// xq[(t * 4 + quad) * nrun + k] (consecutive lanes read consecutive quads),
// then the run sums xs[t * nrun + k].
//
// Waves take groups of PL_ROWS output rows in turn.  A wave walks its work as
// blocks of PL_U runs per lane (lane l of k-block b holds runs
// 64 * (b * PL_U + u) + l) and loads block j + 1 before it computes block j,
// so the next loads are always in flight; the first block is loaded before the
// activations are staged.  At the last k-block of a row group the wave sums
// its lanes and stores the group's outputs.  Rows past c_out (the last group)
// re-read row c_out - 1 and store nothing.
template <int BITS, int NT>
__global__ __launch_bounds__(PL_THREADS) void packed_linear_kernel(
    const uint16_t* __restrict__ X, int n_tok, int64_t c_in, const uint32_t* __restrict__ P,
    int runs_per_group, int group_shift, const float* __restrict__ H, const float* __restrict__ Z,
    const float* __restrict__ bias, int64_t c_out, void* __restrict__ Y, bool y_bf16) {
  extern __shared__ uint4 lds_q[];
  const int nrun = int(c_in / 32);
  float* xs_l = reinterpret_cast<float*>(lds_q + size_t(NT) * 4 * nrun);
  const int lane = threadIdx.x & 63;
  const int64_t nwave = int64_t(gridDim.x) * PL_WAVES;
  const int ng = nrun / runs_per_group;
  const int row_dw = nrun * BITS;
  const int nkb = (nrun + 64 * PL_U - 1) / (64 * PL_U);
  // the two fields of a pair in one dword (4- and 2-bit codes) and the bf16 128.0 pair
  const uint32_t pair_mask = BITS == 4 ? 0x000F000Fu : 0x00030003u;
  const uint32_t magic = BF16_128_PAIR;

  // the group of run k (runs_per_group a power of two: a shift)
  auto group_of = [&](int k) {
    return group_shift >= 0 ? (k >> group_shift) : int(unsigned(k) / unsigned(runs_per_group));
  };
  // Load k-block kb of row group rg (first row rg * PL_ROWS < c_out).
  auto issue = [&](int64_t rg, int kb, uint32_t (&w)[PL_U][PL_ROWS][BITS], float (&hh)[PL_U][PL_ROWS],
                   float (&zz)[PL_U][PL_ROWS]) {
    const uint32_t* prow[PL_ROWS];
    const float *hrow[PL_ROWS], *zrow[PL_ROWS];
#pragma unroll
    for (int r = 0; r < PL_ROWS; ++r) {
      const int64_t row = std::min<int64_t>(rg * PL_ROWS + r, c_out - 1);
      prow[r] = P + row * row_dw;
      hrow[r] = H + row * ng;
      zrow[r] = Z + row * ng;
    }
#pragma unroll
    for (int u = 0; u < PL_U; ++u) {
      const int k = 64 * (kb * PL_U + u) + lane;
      if (k < nrun) {
        const int g = group_of(k);
#pragma unroll
        for (int r = 0; r < PL_ROWS; ++r) {
          load_run<BITS>(prow[r] + k * BITS, w[u][r]);
          hh[u][r] = hrow[r][g];
          zz[u][r] = zrow[r][g];
        }
      }
    }
  };

  float acc[PL_ROWS][NT];
#pragma unroll
  for (int r = 0; r < PL_ROWS; ++r)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[r][t] = 0.f;

  // Compute k-block kb of row group rg from its loaded block; at the last
  // k-block sum the lanes and store the group's outputs.
  auto compute = [&](int64_t rg, int kb, const uint32_t (&w)[PL_U][PL_ROWS][BITS],
                     const float (&hh)[PL_U][PL_ROWS], const float (&zz)[PL_U][PL_ROWS]) {
#pragma unroll
    for (int u = 0; u < PL_U; ++u) {
      const int k = 64 * (kb * PL_U + u) + lane;
      if (k < nrun) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const uint4* xq = lds_q + size_t(t) * 4 * nrun + k;
          uint32_t xp[16];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint4 v = xq[size_t(q) * nrun];
            xp[4 * q] = v.x; xp[4 * q + 1] = v.y; xp[4 * q + 2] = v.z; xp[4 * q + 3] = v.w;
          }
          const float xs = xs_l[t * nrun + k];
#pragma unroll
          for (int r = 0; r < PL_ROWS; ++r) {
            uint32_t cp[16];
            code_pairs<BITS>(w[u][r], cp, pair_mask, magic);
            float p = 0.f;
#pragma unroll
            for (int m = 0; m < 16; ++m) p = dot2_bf16(xp[m], cp[m], p);
            acc[r][t] = __builtin_fmaf(hh[u][r], __builtin_fmaf(-(128.f + zz[u][r]), xs, p), acc[r][t]);
          }
        }
      }
    }
    if (kb == nkb - 1) {
#pragma unroll
      for (int r = 0; r < PL_ROWS; ++r) {
        const int64_t row = rg * PL_ROWS + r;
        const float b = (bias != nullptr && row < c_out) ? bias[row] : 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const float v = wave_sum(acc[r][t]) + b;
          acc[r][t] = 0.f;
          if (lane == 0 && row < c_out && t < n_tok) {
            if (y_bf16)
              static_cast<uint16_t*>(Y)[int64_t(t) * c_out + row] = f2bf(v);
            else
              static_cast<float*>(Y)[int64_t(t) * c_out + row] = v;
          }
        }
      }
    }
  };

  // the wave's blocks in order: row groups wave, wave + nwave, ..., each
  // with k-blocks 0 .. nkb - 1
  int64_t rg = int64_t(blockIdx.x) * PL_WAVES + (threadIdx.x >> 6);
  int kb = 0;
  uint32_t wa[PL_U][PL_ROWS][BITS], wb[PL_U][PL_ROWS][BITS];
  float ha[PL_U][PL_ROWS], za[PL_U][PL_ROWS], hb[PL_U][PL_ROWS], zb[PL_U][PL_ROWS];
  const bool any = rg * PL_ROWS < c_out;
  if (any) issue(rg, kb, wa, ha, za);

  // stage the activation rows: one thread per (token, run)
  for (int idx = threadIdx.x; idx < NT * nrun; idx += PL_THREADS) {
    const int t = idx / nrun, k = idx - t * nrun;
    uint32_t u[16];
    if (t < n_tok) {
      const uint4* src = reinterpret_cast<const uint4*>(X + int64_t(t) * c_in + 32 * int64_t(k));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint4 v = src[e];
        u[4 * e] = v.x; u[4 * e + 1] = v.y; u[4 * e + 2] = v.z; u[4 * e + 3] = v.w;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) u[e] = 0;
    }
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 32; ++j) s += bf2f(uint16_t(u[j >> 1] >> (16 * (j & 1))));
    uint32_t pr[16];
#pragma unroll
    for (int p = 0; p < 16; ++p) {
      const int a = pair_lo<BITS>(p), b = pair_hi<BITS>(p);
      const uint32_t xa = (u[a >> 1] >> (16 * (a & 1))) & 0xffffu;
      const uint32_t xb = (u[b >> 1] >> (16 * (b & 1))) & 0xffffu;
      pr[p] = xa | (xb << 16);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      lds_q[(size_t(t) * 4 + q) * nrun + k] = make_uint4(pr[4 * q], pr[4 * q + 1], pr[4 * q + 2], pr[4 * q + 3]);
    xs_l[t * nrun + k] = s;
  }
  __syncthreads();
  if (!any) return;

  // two load buffers in turn: the next block loads while this one computes
  while (true) {
    int64_t rg2 = kb + 1 < nkb ? rg : rg + nwave;
    int kb2 = kb + 1 < nkb ? kb + 1 : 0;
    bool more = rg2 * PL_ROWS < c_out;
    if (more) issue(rg2, kb2, wb, hb, zb);
    compute(rg, kb, wa, ha, za);
    if (!more) break;
    rg = rg2;
    kb = kb2;
    rg2 = kb + 1 < nkb ? rg : rg + nwave;
    kb2 = kb + 1 < nkb ? kb + 1 : 0;
    more = rg2 * PL_ROWS < c_out;
    if (more) issue(rg2, kb2, wa, ha, za);
    compute(rg, kb, wb, hb, zb);
    if (!more) break;
    rg = rg2;
    kb = kb2;
  }
}

// Global -> LDS copies of 16 or 4 bytes per lane: lane l's bytes land at LDS
// byte address lds + size l.  Inline assembly, so the compiler neither waits
// for them nor counts them: the kernel waits itself (wait_vm).  m0 (the copy's
// LDS base) is saved and restored, with one wait state before the copy.
OQ_DEV void copy16_lds(const void* base, uint32_t off, uint32_t lds) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds);
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %2, %3\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(m0v), "v"(off), "s"(base)
      : "memory");
}
OQ_DEV void copy4_lds(const void* base, uint32_t off, uint32_t lds) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds);
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dword %2, %3\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(m0v), "v"(off), "s"(base)
      : "memory");
}
// the same copy from a full address per lane
OQ_DEV void copy4_lds_v(uint64_t addr, uint32_t lds) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds);
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dword %2, off\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(m0v), "v"(addr)
      : "memory");
}
// until at most N of the wave's memory operations are outstanding
template <int N>
OQ_DEV void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory");
}
// until the wave's LDS reads have their data: before a copy into a slot that they
// read (the compiler would let a read's value arrive after the copy is issued)
OQ_DEV void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
OQ_DEV uint32_t lds_addr(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
      (__attribute__((address_space(3))) const char*)(p)));
}

// ------------------------------------------------------------------ up to 32 tokens
// A workgroup takes tiles of 16 RT output rows in turn (blockIdx, + gridDim, ..)
// and its eight waves the 256-channel super-blocks wave, wave + 8, ... of K,
// two 128-channel blocks each.  For a block, lane (f, i) (f = lane / 16, i =
// lane % 16) takes run f of output row i of each 16-row tile; matrix
// instruction m (0..3) multiplies the tokens (A operand, 16 a tile) by codes
// 4 m .. 4 m + 3 and 16 + 4 m .. of every lane's run widened to 2^BITS + q (B
// operand).  A product of the same activations with ones gives xs = sum x, and
// a block adds h (p - (2^BITS + z) xs) to each output, in fp32.
//
// SUB = 1, 2 or 4 parts per block, for groups of whole 128-, 64- or
// 32-channel parts: part j's product takes the activations of the other
// parts' lanes as zeros.
//
// What bounds it at few tokens is the stream of codes: everything a wave reads
// goes global -> LDS by asynchronous copies into a ring of its own (no
// registers, no barriers), D units deep and across tiles, so the loads never
// wait for the arithmetic.  A copy instruction takes whole consecutive 16-byte
// chunks of rows (read by lanes in operand order, every four neighbouring
// lanes would touch four rows).  A unit is a super-block (up to 4 tokens) or a
// block (more) of codes with its step sizes and zero points, and for more than
// 4 tokens its activations; up to 4 tokens the wave's whole share of the
// activations is copied once.  In LDS chunk c of row r sits at c ^ swz(r), so
// the lanes of one operand read hit distinct banks.
//
// The waves' partial outputs are added through LDS, the even waves' and the odd
// waves' in order and then the two sums, as the tiled kernel adds them; a token's
// sums depend neither on the other tokens of its batch nor on RT.
constexpr int PM_THREADS = 512;
constexpr int PM_WAVES = PM_THREADS / 64;
constexpr int PM_BLOCK = 128;                  // channels of a K block
constexpr int PM_RED_PITCH = 17;
constexpr int PM_BIAS_TILES = 64;              // tiles a workgroup may take with a bias

template <int BITS, int TT, int RT, int SUB>
struct MfmaCfg {
  static constexpr bool KEEP = TT == 4;
  static constexpr int UB = KEEP ? 2 : 1;                  // blocks of a unit
  static constexpr int ROWB = UB * 16 * BITS;              // a unit's bytes of one row
  static constexpr int WB = 16 * RT * ROWB;
  static constexpr int HZ = 2 * 16 * RT * UB * SUB;        // step sizes and zero points
  static constexpr int XB = KEEP ? 0 : TT * 256;
  static constexpr int SLOT = WB + HZ * 4 + XB;            // ring slot, bytes
  static constexpr int RED = PM_WAVES * RT * (TT < 16 ? TT : 16) * PM_RED_PITCH * 4;
  static constexpr int NRED = TT > 16 ? 1 : 2;             // partial-output buffers
  // whether a workgroup can run at all: two-slot rings and partial outputs in LDS
  static constexpr bool FITS = size_t(PM_WAVES) * 2 * SLOT + size_t(NRED) * RED <= PL_LDS_MAX;
  // LDS of the workgroup: rings, kept activations, partial outputs, biases
  static size_t lds(int depth, int64_t c_in, int n_tok, bool bias) {
    const size_t sb = size_t((c_in + 255) / 256);
    const size_t keep = KEEP ? (sb + PM_WAVES - 1) / PM_WAVES * PM_WAVES * size_t(n_tok) * 512 : 0;
    return size_t(PM_WAVES) * depth * SLOT + keep + size_t(NRED) * RED +
           (bias ? size_t(PM_BIAS_TILES) * 16 * RT * 4 : 0);
  }
};

// TT: tokens staged (4, 8, 16, 24 or 32).  A16: rows of whole 16-byte chunks (c_in a
// multiple of 128), else dword copies.
template <int BITS, int TT, int RT, int SUB, int D, bool A16>
__global__ __launch_bounds__(PM_THREADS) void packed_mfma_kernel(
    const uint16_t* __restrict__ X, int n_tok, int64_t c_in, const uint32_t* __restrict__ packed,
    int ng, uint32_t group_inv, const float* __restrict__ H, const float* __restrict__ Z,
    const float* __restrict__ bias, int64_t c_out, void* __restrict__ Y, bool y_bf16, int ntile) {
  using Cfg = MfmaCfg<BITS, TT, RT, SUB>;
  constexpr bool KEEP = Cfg::KEEP;
  constexpr int UB = Cfg::UB, ROWB = Cfg::ROWB, SLOT = Cfg::SLOT;
  constexpr int NTB = (TT + 15) / 16;          // token tiles of 16
  constexpr int CB = A16 ? 16 : 4;             // bytes of a copied chunk
  constexpr int RC = ROWB / CB;                // chunks of a row
  constexpr int NW = (16 * RT * RC + 63) / 64; // copies of a unit: codes,
  constexpr int NH = (Cfg::HZ + 63) / 64;      // step sizes and zero points,
  constexpr int NX = KEEP ? 0 : TT / 4;        // activations
  constexpr int NU = NW + NH + NX;
  static_assert((D - 1) * NU < 64, "vmcnt range");
  // chunk swizzle of codes whose row pitch puts rows on the same banks
  constexpr bool SWZ = A16 && (BITS == 2 || BITS == 4);
  extern __shared__ uint4 lds_q[];
  char* lds0 = reinterpret_cast<char*>(lds_q);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: scalar addresses
  const int f = lane >> 4, i = lane & 15;
  const int nrun = int(c_in / 32), nsb = (nrun + 7) / 8, nblk = (nrun + 3) / 4;
  const int nk = nsb > wave ? (nsb - wave + PM_WAVES - 1) / PM_WAVES : 0;   // the wave's super-blocks
  const int kmax = (nsb + PM_WAVES - 1) / PM_WAVES;
  const int grid = gridDim.x;
  const int mytiles = (ntile - int(blockIdx.x) + grid - 1) / grid;
  char* ring = lds0 + wave * (D * SLOT);
  char* keep0 = lds0 + PM_WAVES * D * SLOT;
  char* keep = keep0 + size_t(wave) * kmax * n_tok * 512;
  float* red0 = reinterpret_cast<float*>(keep0 + (KEEP ? size_t(PM_WAVES) * kmax * n_tok * 512 : 0));
  float* sbias = red0 + Cfg::NRED * Cfg::RED / 4;
  const uint32_t ring_a = lds_addr(ring);
  const uint32_t rowb = uint32_t(nrun * BITS * 4);
  const CodeMasks<BITS> cm;
  constexpr float OFF = float(1 << BITS);
  const bf16x8_t ones = __builtin_bit_cast(bf16x8_t, make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));
  auto swz = [](int r) {
    constexpr int NCH = ROWB / 16;             // 16-byte chunks of a row
    return SWZ ? (r / (256 / ROWB)) & (NCH - 1) : 0;
  };

  // Copies of unit (tile, block b0 .. b0 + UB - 1) into ring slot `s`.  Rows
  // past c_out and chunks past a row's end re-read the last one.
  uint32_t wcol[NW], wrow[NW];                 // a lane's chunk: column bytes in the unit, row
#pragma unroll
  for (int j = 0; j < NW; ++j) {
    const int id = 64 * j + lane, c = id % RC;
    wrow[j] = uint32_t(id / RC);
    wcol[j] = uint32_t(CB * (c ^ swz(int(wrow[j]) & 15)));
  }
  auto issue = [&](int tile, int b0, int s) {
    const int64_t ot = int64_t(tile) * (16 * RT);
    const uint32_t last = uint32_t(c_out - ot < 16 * RT ? c_out - ot - 1 : 16 * RT - 1);
    uint32_t dst = ring_a + uint32_t(s * SLOT);
    const char* wbase = reinterpret_cast<const char*>(packed) + ot * rowb;
    const uint32_t col0 = uint32_t(b0 * 16 * BITS);
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      const uint32_t off = __umul24(min(wrow[j], last), rowb) + min(col0 + wcol[j], rowb - CB);
      if (64 * NW == 16 * RT * RC || 64 * j + lane < 16 * RT * RC) {
        if constexpr (A16) copy16_lds(wbase, off, dst + 1024 * j);
        else copy4_lds(wbase, off, dst + 256 * j);
      }
    }
    dst += Cfg::WB;
    const float *hb = H + ot * ng, *zb = Z + ot * ng;
#pragma unroll
    for (int j = 0; j < NH; ++j) {
      // h of every row first, then z: [2][16 RT][UB SUB]
      constexpr int HALF = Cfg::HZ / 2;
      const int id = 64 * j + lane, e = id % HALF;
      const uint32_t row = uint32_t(e / (UB * SUB));
      const int part = 4 * b0 + (4 / SUB) * (e % (UB * SUB));
      const uint32_t off = 4 * (__umul24(min(row, last), uint32_t(ng)) +
                                uint32_t(group_of(part < nrun ? part : nrun - 1, group_inv)));
      if constexpr (HALF >= 64) {
        copy4_lds(64 * j < HALF ? hb : zb, off, dst + 256 * j);
      } else {
        // a copy of both: its lanes address h, and z from there
        const uint64_t a = reinterpret_cast<uint64_t>(id < HALF ? hb : zb) + off;
        if (Cfg::HZ % 64 == 0 || id < Cfg::HZ) copy4_lds_v(a, dst + 256 * j);
      }
    }
    dst += Cfg::HZ * 4;
    if constexpr (!KEEP) {
#pragma unroll
      for (int j = 0; j < NX; ++j) {
        const int t = 4 * j + (lane >> 4), c = (lane & 15) ^ (t & 15);
        const uint32_t col = uint32_t(b0 * 256 + 16 * c);
        const uint32_t off = uint32_t(min(t, n_tok - 1)) * uint32_t(c_in * 2) + min(col, uint32_t(c_in * 2 - 16));
        copy16_lds(X, off, dst + 1024 * j);
      }
    }
  };

  f32x4_t y[RT][NTB];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int tb = 0; tb < NTB; ++tb) y[rt][tb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // block b (the u-th of its unit) from ring slot `s`; xrow: this lane's
  // token row of the block's activations, per token tile
  auto compute = [&](int b, int ub, const char* slot, const char* xb, uint32_t xstride) {
    bf16x8_t xf[NTB][4];
    const bool tail = !A16 && 4 * b + 4 > nrun;        // uniform
#pragma unroll
    for (int tb = 0; tb < NTB; ++tb) {
      const int t = KEEP ? min(i & 3, n_tok - 1) : min(16 * tb + i, TT - 1);
      const char* xr = xb + uint32_t(t) * xstride;
      if constexpr (KEEP) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
          xf[tb][m] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(xr + 16 * ((4 * f + m) ^ t)));
        continue;
      }
#pragma unroll
      for (int mm = 0; mm < 2; ++mm) {
        uint4 lo = *reinterpret_cast<const uint4*>(xr + 16 * ((4 * f + mm) ^ (t & 15)));
        uint4 hi = *reinterpret_cast<const uint4*>(xr + 16 * ((4 * f + 2 + mm) ^ (t & 15)));
        uint4 u0, u1;
        interleave_x(lo, hi, u0, u1);
        if (tail && 4 * b + f >= nrun) u0 = u1 = make_uint4(0u, 0u, 0u, 0u);
        xf[tb][2 * mm] = __builtin_bit_cast(bf16x8_t, u0);
        xf[tb][2 * mm + 1] = __builtin_bit_cast(bf16x8_t, u1);
      }
    }
    uint32_t R[RT][BITS];
    float hh[RT][SUB], nz[RT][SUB];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      uint32_t w[BITS];
      const int row = 16 * rt + i;
      const char* wr = slot + row * ROWB;
      if constexpr (SWZ) {
        // the run's bytes: 4 BITS at (4 ub + f) runs, in 16-byte chunks
        const int at = (4 * ub + f) * 4 * BITS;
        load_run<BITS>(reinterpret_cast<const uint32_t*>(wr + 16 * ((at >> 4) ^ swz(i)) + (at & 15)), w);
      } else {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(wr) + (4 * ub + f) * BITS;
#pragma unroll
        for (int k = 0; k < BITS; ++k) w[k] = src[k];
      }
      interleave_run<BITS>(w, R[rt]);
      const float* hz = reinterpret_cast<const float*>(slot + Cfg::WB) + row * (UB * SUB) + ub * SUB;
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
        hh[rt][u] = hz[u];
        nz[rt][u] = -(OFF + hz[Cfg::HZ / 2 + u]);
      }
    }
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
      bf16x8_t xa[NTB][4];
      const bool mine = SUB == 1 || f / (4 / SUB) == u;
      f32x4_t xs[NTB];
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb) {
        xs[tb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          if constexpr (SUB > 1) {
            const uint4 v = __builtin_bit_cast(uint4, xf[tb][m]);
            xa[tb][m] = __builtin_bit_cast(
                bf16x8_t, make_uint4(mine ? v.x : 0u, mine ? v.y : 0u, mine ? v.z : 0u, mine ? v.w : 0u));
          } else {
            xa[tb][m] = xf[tb][m];
          }
          xs[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[tb][m], ones, xs[tb], 0, 0, 0);
        }
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        f32x4_t acc[NTB];
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) acc[tb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const bf16x8_t q = code_frag<BITS>(R[rt], m, cm);
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb)
            acc[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[tb][m], q, acc[tb], 0, 0, 0);
        }
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            y[rt][tb][r] = __builtin_fmaf(hh[rt][u], __builtin_fmaf(nz[rt][u], xs[tb][r], acc[tb][r]), y[rt][tb][r]);
      }
      if constexpr (SUB > 1) __builtin_amdgcn_sched_barrier(0);   // one part's registers at a time
    }
  };

  // a tile's end: the waves' partial outputs (lane (f, i) holds tokens 16 tb +
  // 4 f + r of row 16 rt + i) meet in LDS, one token tile at a time.  With two
  // buffers a wave can be one barrier ahead of the readers of the other.
  constexpr int RTT = TT < 16 ? TT : 16;       // tokens of a buffer
  int rbuf = 0;
  auto finish = [&](int tile, int nth) {
#pragma unroll
    for (int tb = 0; tb < NTB; ++tb) {
      float* red = red0 + rbuf * (Cfg::RED / 4);   // [PM_WAVES][RT][RTT][PITCH]
      if (Cfg::NRED == 2) rbuf ^= 1;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int t = 4 * f + r;
          if (t < RTT) red[((wave * RT + rt) * RTT + t) * PM_RED_PITCH + i] = y[rt][tb][r];
          y[rt][tb][r] = 0.f;
        }
      lds_barrier();
      for (int e = tid; e < 16 * RT * RTT; e += PM_THREADS) {
        const int t = e / (16 * RT), oo = e % (16 * RT), rt = oo >> 4, ii = oo & 15;
        const int64_t o = int64_t(tile) * (16 * RT) + oo;
        if (16 * tb + t < n_tok && o < c_out) {
          float p[2] = {0.f, 0.f};             // even and odd waves
#pragma unroll
          for (int w = 0; w < PM_WAVES; ++w) p[w & 1] += red[((w * RT + rt) * RTT + t) * PM_RED_PITCH + ii];
          float v = p[0] + p[1];
          if (bias) v += sbias[nth * (16 * RT) + oo];
          const int64_t at = int64_t(16 * tb + t) * c_out + o;
          if (y_bf16) static_cast<uint16_t*>(Y)[at] = f2bf(v);
          else static_cast<float*>(Y)[at] = v;
        }
      }
      if (Cfg::NRED == 1) lds_barrier();
    }
  };

  // this workgroup's biases, all tiles (the host bounds their number)
  if (bias) {
    for (int e = tid; e < mytiles * 16 * RT; e += PM_THREADS) {
      const int64_t o = (int64_t(blockIdx.x) + int64_t(e / (16 * RT)) * grid) * (16 * RT) + e % (16 * RT);
      sbias[e] = o < c_out ? bias[o] : 0.f;
    }
  }
  if (nk == 0) {                               // K is shorter than the waves
    for (int n = 0; n < mytiles; ++n) finish(int(blockIdx.x) + n * grid, n);
    return;
  }
  // x / n_tok for the small x of the kept activations (n_tok 1..4, x < 16384)
  const int tok_inv = (65536 + n_tok - 1) / n_tok;
  auto tok_div = [&](int x) { return (x * tok_inv) >> 16; };
  if constexpr (KEEP) {
    // [k][block of 2][token][256 bytes], chunk c of token t at c ^ t
    const uint32_t ka = lds_addr(keep);
    const int total = nk * n_tok * 32;
    for (int c0 = 0; c0 < total; c0 += 64) {
      const int id = c0 + lane, bt = id >> 4, kb = tok_div(bt), t = bt - kb * n_tok, c = (id & 15) ^ t;
      const uint32_t col = uint32_t((wave + PM_WAVES * (kb >> 1)) * 512 + (kb & 1) * 256 + 16 * c);
      const uint32_t off = uint32_t(t) * uint32_t(c_in * 2) + min(col, uint32_t(c_in * 2 - 16));
      if (id < total) copy16_lds(X, off, ka + uint32_t(c0 * 16));
    }
  }
  // the walk over the wave's units: (tile, k-th super-block, block of it)
  constexpr int BPS = 2 / UB;                  // units of a super-block
  int tile2 = blockIdx.x, k2 = 0, h2 = 0, left = mytiles * nk * BPS;   // units to issue
  auto prefetch = [&](int s) {
    issue(tile2, 2 * (wave + PM_WAVES * k2) + h2, s);
    --left;
    if (++h2 == BPS) {
      h2 = 0;
      if (++k2 == nk) { k2 = 0; tile2 += grid; }
    }
  };
  int inflight = 0;
#pragma unroll
  for (int s = 0; s < D; ++s)
    if (left > 0) { prefetch(s); ++inflight; }
  if constexpr (KEEP) {
    // the kept activations (older than the units) into the codes' pair order,
    // in place; runs past the end of K become zeros
    if (inflight == D) wait_vm<D * NU>();
    else wait_vm<0>();
    const int total = nk * n_tok * 16;         // (k, block, token, run, half) per lane
    for (int c0 = 0; c0 < total; c0 += 64) {
      const int id = c0 + lane, bt = id >> 3, run = (id >> 1) & 3, half = id & 1;
      const int kb = tok_div(bt), t = bt - kb * n_tok;
      char* row = keep + (size_t(kb) * n_tok + t) * 256;
      const int c = 4 * run + half, r = 4 * (2 * (wave + PM_WAVES * (kb >> 1)) + (kb & 1)) + run;
      uint4 lo = make_uint4(0u, 0u, 0u, 0u), hi = lo, u0, u1;
      if (id < total && r < nrun) {
        lo = *reinterpret_cast<const uint4*>(row + 16 * (c ^ t));
        hi = *reinterpret_cast<const uint4*>(row + 16 * ((c + 2) ^ t));
      }
      interleave_x(lo, hi, u0, u1);
      wave_lds_order();                        // a run's two lanes read before they write
      if (id < total) {
        const int d = 4 * run + 2 * half;
        *reinterpret_cast<uint4*>(row + 16 * (d ^ t)) = u0;
        *reinterpret_cast<uint4*>(row + 16 * ((d + 1) ^ t)) = u1;
      }
    }
    wave_lds_order();
  }
  int s = 0;
  for (int n = 0; n < mytiles; ++n) {
    const int tile = int(blockIdx.x) + n * grid;
    for (int k = 0; k < nk; ++k)
      for (int hf = 0; hf < BPS; ++hf) {
        // the oldest unit (and, before it, the kept activations) has landed
        if (inflight == D) wait_vm<(D - 1) * NU>();
        else wait_vm<0>();
        const char* slot = ring + s * SLOT;
        const int b0 = 2 * (wave + PM_WAVES * k) + hf;
#pragma unroll
        for (int ub = 0; ub < UB; ++ub)
          if (KEEP || b0 + ub < nblk)           // KEEP: a missing block's activations are zeros
            compute(b0 + ub, ub, slot, KEEP ? keep + size_t(2 * k + ub) * n_tok * 256 : slot + Cfg::WB + Cfg::HZ * 4, 256);
        if (left > 0) {
          wait_lds_reads();
          prefetch(s);
        } else {
          --inflight;
        }
        s = s + 1 == D ? 0 : s + 1;
      }
    finish(tile, n);
  }
}

// ------------------------------------------------------------------ 17 to 32 tokens, many rows
// The small-batch kernel's product where the rings of 32 tokens leave LDS no room
// for two row tiles (or, with 6- and 7-bit codes, for one): only the activations
// go through LDS, a block ahead, and a lane's codes, step size and zero point
// through registers.  Groups of whole blocks; shares of K, arithmetic and order of
// the sums are the small-batch kernel's, so the outputs are the same bits.
// (W6, 32 tokens, 24576 x 8192: 110 us in launches of 24 and 8, 76 here.)
constexpr int PW_TOKENS = 32;

template <int BITS, int RT>
__global__ __launch_bounds__(PM_THREADS) void packed_wide_kernel(
    const uint16_t* __restrict__ X, int n_tok, int64_t c_in, const uint32_t* __restrict__ packed,
    int ng, uint32_t group_inv, const float* __restrict__ H, const float* __restrict__ Z,
    const float* __restrict__ bias, int64_t c_out, void* __restrict__ Y, bool y_bf16) {
  constexpr int NTB = 2, XB = PW_TOKENS * 256;   // bytes of a block's activations
  extern __shared__ uint4 lds_q[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int f = lane >> 4, i = lane & 15;
  const int nrun = int(c_in / 32), nsb = (nrun + 7) / 8, nblk = nrun / 4;
  const int64_t o0 = int64_t(blockIdx.x) * (16 * RT);
  char* ring = reinterpret_cast<char*>(lds_q) + wave * (2 * XB);
  const uint32_t ring_a = lds_addr(ring);
  const CodeMasks<BITS> cm;
  constexpr float OFF = float(1 << BITS);
  const bf16x8_t ones = __builtin_bit_cast(bf16x8_t, make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));
  // this lane's rows (rows past c_out re-read the last one and store nothing)
  const uint32_t* prow[RT];
  const float *hrow[RT], *zrow[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int64_t row = std::min<int64_t>(o0 + 16 * rt + i, c_out - 1);
    prow[rt] = packed + (row * nrun + f) * BITS;
    hrow[rt] = H + row * ng;
    zrow[rt] = Z + row * ng;
  }
  // block b's activations into buffer `s`: a copy takes four tokens' 256 bytes,
  // chunk c of token t at c ^ (t % 16); tokens past n_tok re-read the last one
  auto copy_x = [&](int b, int s) {
#pragma unroll
    for (int j = 0; j < PW_TOKENS / 4; ++j) {
      if (4 * j >= n_tok) break;               // uniform
      const int t = 4 * j + f, c = i ^ (t & 15);
      const uint32_t off = uint32_t(min(t, n_tok - 1)) * uint32_t(c_in * 2) + uint32_t(b * 256 + 16 * c);
      copy16_lds(X, off, ring_a + uint32_t(s * XB + 1024 * j));
    }
  };
  uint32_t wn[RT][BITS];
  float hn[RT], zn[RT];
  auto load_w = [&](int b) {
    const int g = group_of(4 * b, group_inv);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      load_run<BITS>(prow[rt] + b * (4 * BITS), wn[rt]);
      hn[rt] = hrow[rt][g];
      zn[rt] = zrow[rt][g];
    }
  };
  // the wave's blocks: both of super-blocks wave, wave + 8, ..
  auto next = [&](int b) { return b & 1 ? b + 2 * PM_WAVES - 1 : b + 1; };

  f32x4_t y[RT][NTB];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int tb = 0; tb < NTB; ++tb) y[rt][tb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  int b = 2 * wave, s = 0;
  if (b < nblk) {
    copy_x(b, 0);
    load_w(b);
  }
  for (; b < nblk; s ^= 1) {
    wait_vm<0>();                              // block b, issued one turn ago, has landed
    uint32_t R[RT][BITS];
    float hh[RT], nz[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      interleave_run<BITS>(wn[rt], R[rt]);
      hh[rt] = hn[rt];
      nz[rt] = -(OFF + zn[rt]);
    }
    // (the last block of K may be the first of its super-block)
    const int b2 = next(b);
    if (b2 < nblk) {
      wait_lds_reads();                        // the buffer's former block has been read
      copy_x(b2, s ^ 1);
      load_w(b2);
    }
    f32x4_t acc[RT][NTB], xs[NTB];
#pragma unroll
    for (int tb = 0; tb < NTB; ++tb) {
      xs[tb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt][tb] = xs[tb];
    }
    const char* xb = ring + s * XB + i * 256;
    bf16x8_t xf[NTB][4];
#pragma unroll
    for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
      for (int mm = 0; mm < 2; ++mm) {
        uint4 u0, u1;
        interleave_x(*reinterpret_cast<const uint4*>(xb + tb * 4096 + 16 * ((4 * f + mm) ^ i)),
                     *reinterpret_cast<const uint4*>(xb + tb * 4096 + 16 * ((4 * f + 2 + mm) ^ i)), u0, u1);
        xf[tb][2 * mm] = __builtin_bit_cast(bf16x8_t, u0);
        xf[tb][2 * mm + 1] = __builtin_bit_cast(bf16x8_t, u1);
      }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb)
        xs[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[tb][m], ones, xs[tb], 0, 0, 0);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const bf16x8_t q = code_frag<BITS>(R[rt], m, cm);
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb)
          acc[rt][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[tb][m], q, acc[rt][tb], 0, 0, 0);
      }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          y[rt][tb][r] = __builtin_fmaf(hh[rt], __builtin_fmaf(nz[rt], xs[tb][r], acc[rt][tb][r]), y[rt][tb][r]);
    b = b2;
  }
  // the waves' partial outputs (lane (f, i): tokens 16 tb + 4 f + r of row 16 rt +
  // i) take the buffers' place: every copy has landed and been read
  __syncthreads();
  float* red = reinterpret_cast<float*>(lds_q);   // [PM_WAVES][RT][32 tokens][PITCH]
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        red[((wave * RT + rt) * PW_TOKENS + 16 * tb + 4 * f + r) * PM_RED_PITCH + i] = y[rt][tb][r];
  __syncthreads();
  for (int e = tid; e < 16 * RT * PW_TOKENS; e += PM_THREADS) {
    const int t = e / (16 * RT), oo = e % (16 * RT), rt = oo >> 4, ii = oo & 15;
    const int64_t o = o0 + oo;
    if (t < n_tok && o < c_out) {
      float p[2] = {0.f, 0.f};                 // even and odd waves
#pragma unroll
      for (int w = 0; w < PM_WAVES; ++w) p[w & 1] += red[((w * RT + rt) * PW_TOKENS + t) * PM_RED_PITCH + ii];
      const float v = p[0] + p[1] + (bias ? bias[o] : 0.f);
      const int64_t at = int64_t(t) * c_out + o;
      if (y_bf16) static_cast<uint16_t*>(Y)[at] = f2bf(v);
      else static_cast<float*>(Y)[at] = v;
    }
  }
}

// ------------------------------------------------------------------ prompts
// The same product as a tiled one for many tokens.  A workgroup of eight waves
// owns 128 outputs x 16 NTB tokens: wave w takes outputs 32 (w % 4) .. + 31 (two
// 16-row tiles, codes straight from global memory into registers) and K block
// 2 it + w / 4 of iteration it.  The activations of an iteration's two blocks
// are staged once for all waves, double-buffered, in the codes' pair order with
// the slots swizzled as above.  The two K halves are added through LDS at the end.
//
// Groups of whole blocks (SAME): a token's outputs are the small-batch kernel's
// bit for bit, so they do not change with the size of its batch.  xs is the same
// product with ones, and waves w / 4 = 0 and 1 take the even and the odd
// super-blocks in the order of the small-batch kernel's waves (0, 8, .., then 2,
// 10, ..; 1, 9, ..), each wave's share summed on its own.  It costs: with xs
// from the staging thread and K in sequence, 500 tokens through a 7B block's
// linears at W4 took 445 us, now 450 to 460 (2048 tokens, 12288 x 4096, W3: 403 -> 446).
// Shares of contiguous super-blocks cost more in the small-batch kernel (W2 g64,
// 4 tokens: 257 -> 300 us); sums formed by one wave for the others were no faster
// (495 us).
//
// Other groups: the thread that interleaves the activations also sums them (xs
// per token and part), so the matrix cores run only the products, and K goes in
// sequence.
constexpr int PT_N = 128;                      // outputs per workgroup
template <int NTB, int SUB>
constexpr size_t tile_lds() {
  const size_t x = size_t(2) * 16 * NTB * 512 + size_t(2) * 2 * SUB * 16 * NTB * sizeof(float);
  const size_t r = size_t(4) * 2 * 16 * NTB * PM_RED_PITCH * sizeof(float);
  return x > r ? x : r;
}

template <int BITS, int NTB, int SUB>
__global__ __launch_bounds__(PM_THREADS) void packed_tile_kernel(
    const uint16_t* __restrict__ X, int n_tok, int64_t c_in, const uint32_t* __restrict__ packed,
    int ng, uint32_t group_inv, const float* __restrict__ H, const float* __restrict__ Z,
    const float* __restrict__ bias, int64_t c_out, void* __restrict__ Y, bool y_bf16, int ntt) {
  constexpr int TM = 16 * NTB;                 // tokens
  constexpr int XR = TM * 16 / PM_THREADS;     // staging rounds (32 tokens each)
  constexpr bool SAME = SUB == 1;              // sums in the small-batch kernel's order
  constexpr int KSTEP = SAME ? 2 : 1;          // blocks from kw 0's to kw 1's
  extern __shared__ uint4 lds_q[];
  char* xb = reinterpret_cast<char*>(lds_q);   // [2 buffers][TM][2 blocks][256 bytes]
  float* xsb = reinterpret_cast<float*>(xb + size_t(2) * TM * 512);   // [2][2 blocks][SUB][TM]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int f = lane >> 4, i = lane & 15;
  const int wn = wave & 3, kw = wave >> 2;
  // XCD x takes a contiguous range of tiles, token tiles fastest: the tiles
  // that read the same codes run together on one L2
  const int nb = gridDim.x, xcd = blockIdx.x & 7, q8 = nb >> 3, rem = nb & 7;
  const int L = xcd * q8 + min(xcd, rem) + (blockIdx.x >> 3);
  const int t0 = (L % ntt) * TM;
  const int64_t o0 = int64_t(L / ntt) * PT_N + 32 * wn;
  const int nrun = int(c_in / 32), nblk = (nrun + 3) / 4, nsb = (nrun + 7) / 8;
  const int nit = SAME ? 2 * ((nsb + 1) / 2) : (nblk + 1) / 2;
  const CodeMasks<BITS> cm;
  constexpr float OFF = float(1 << BITS);
  const bf16x8_t ones = __builtin_bit_cast(bf16x8_t, make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));
  // The walk over K: `b` is kw 0's block.  SAME: the blocks of super-blocks 0, 8,
  // .. (kw 1: of the next ones), then of 2, 10, .. and so on.  True where a share
  // ends.
  auto next = [&](int& b) {
    if (!SAME) {
      b += 2;
      return false;
    }
    if (!(b & 1)) {
      ++b;
      return false;
    }
    b += 2 * PM_WAVES - 1;
    if (b < 2 * nsb) return false;
    b = 2 * (((b >> 1) & (PM_WAVES - 1)) + 2);
    return true;
  };

  // tokens and rows past the end read zeros (and store nothing); iterations
  // past the last read nothing
  constexpr uint32_t NONE = 0x80000000u;
  const int mt = min(TM, n_tok - t0);
  const rsrc_t rx = make_rsrc(X + int64_t(t0) * c_in, uint32_t(mt) * uint32_t(c_in * 2));
  const int64_t left = c_out - o0;
  const uint32_t rows = left <= 0 ? 0u : left < 32 ? uint32_t(left) : 32u;
  const rsrc_t rw = make_rsrc(packed + o0 * nrun * BITS, rows * uint32_t(nrun * BITS * 4));
  const rsrc_t rh = make_rsrc(H + o0 * ng, rows * uint32_t(ng * 4)), rz = make_rsrc(Z + o0 * ng, rows * uint32_t(ng * 4));
  // staging: 16 threads per token, thread (run 0..7 of the iteration, half)
  const int srun = (tid >> 1) & 7, shalf = tid & 1, st0 = tid >> 4;
  const uint32_t xoff = uint32_t(st0) * uint32_t(c_in * 2) + uint32_t(256 * KSTEP * (srun >> 2) + 64 * (srun & 3) + 16 * shalf);
  const uint32_t woff = __umul24(uint32_t(i), uint32_t(nrun * BITS * 4)) + uint32_t(f * BITS * 4);
  const uint32_t goff = __umul24(uint32_t(i), uint32_t(ng * 4));

  uint4 slo[XR], shi[XR];
  uint32_t wn_[2][BITS], hn[2][SUB], zn[2][SUB];
  int bx = 0, bw = 0, bs = 0, bc = 0;           // blocks to load, to load codes of, to stage, to compute
  auto issue_x = [&](bool any) {
#pragma unroll
    for (int j = 0; j < XR; ++j) {
      const uint32_t o = any ? xoff + uint32_t(32 * j) * uint32_t(c_in * 2) + uint32_t(256 * bx) : NONE;
      buffer_load<4>(rx, o, reinterpret_cast<uint32_t*>(&slo[j]));
      buffer_load<4>(rx, o + 32, reinterpret_cast<uint32_t*>(&shi[j]));
    }
    next(bx);
  };
  auto issue_w = [&](bool any) {
    const int b = any ? bw + KSTEP * kw : nblk;
    next(bw);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const uint32_t wr = 16 * rt * uint32_t(nrun * BITS * 4), gr = 16 * rt * uint32_t(ng * 4);
      buffer_load<BITS>(rw, b < nblk ? woff + wr + uint32_t(4 * b * BITS * 4) : NONE, wn_[rt]);
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
        const int part = 4 * b + (4 / SUB) * u;
        const uint32_t g = part < nrun ? goff + gr + uint32_t(4 * group_of(part, group_inv)) : NONE;
        buffer_load<1>(rh, g, &hn[rt][u]);        // zeros: no such part
        buffer_load<1>(rz, g, &zn[rt][u]);
      }
    }
  };
  auto stage = [&](int buf) {
    const int blk = srun >> 2;
    const bool miss = 4 * (bs + KSTEP * blk) + (srun & 3) >= nrun;
    next(bs);
    const int c = 4 * (srun & 3) + 2 * shalf;
#pragma unroll
    for (int j = 0; j < XR; ++j) {
      const int t = st0 + 32 * j;
      uint4 u0, u1;
      interleave_x(slo[j], shi[j], u0, u1);
      if (miss) u0 = u1 = make_uint4(0u, 0u, 0u, 0u);
      char* row = xb + (size_t(buf) * TM + t) * 512 + blk * 256;
      *reinterpret_cast<uint4*>(row + 16 * (c ^ (t & 15))) = u0;
      *reinterpret_cast<uint4*>(row + 16 * ((c + 1) ^ (t & 15))) = u1;
      if constexpr (SAME) continue;
      // this thread's 16 channels, then the part's lanes (8 / SUB of them)
      float s0 = 0.f, s1 = 0.f;
      s0 = dot2_bf16(u0.x, 0x3f803f80u, s0); s1 = dot2_bf16(u1.x, 0x3f803f80u, s1);
      s0 = dot2_bf16(u0.y, 0x3f803f80u, s0); s1 = dot2_bf16(u1.y, 0x3f803f80u, s1);
      s0 = dot2_bf16(u0.z, 0x3f803f80u, s0); s1 = dot2_bf16(u1.z, 0x3f803f80u, s1);
      s0 = dot2_bf16(u0.w, 0x3f803f80u, s0); s1 = dot2_bf16(u1.w, 0x3f803f80u, s1);
      float s = s0 + s1;
      s += dpp_f(s, 0);
      if constexpr (SUB <= 2) s += dpp_f(s, 1);
      if constexpr (SUB == 1) s += dpp_f(s, 2);
      if ((lane & (8 / SUB - 1)) == 0)
        xsb[((buf * 2 + blk) * SUB + (SUB == 1 ? 0 : (srun & 3) / (4 / SUB))) * TM + t] = s;
    }
  };

  f32x4_t y[2][NTB], total[2][NTB];            // the current share's, the finished shares'
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int tb = 0; tb < NTB; ++tb) y[rt][tb] = total[rt][tb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto end_share = [&]() {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb) {
        total[rt][tb] += y[rt][tb];
        y[rt][tb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      }
  };

  issue_x(true);
  issue_w(true);
  stage(0);
  issue_x(true);
  lds_barrier();
  for (int it = 0; it < nit; ++it) {
    const int buf = it & 1;
    uint32_t R[2][BITS];
    float hh[2][SUB], nz[2][SUB];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      interleave_run<BITS>(wn_[rt], R[rt]);
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
        hh[rt][u] = __uint_as_float(hn[rt][u]);
        nz[rt][u] = -(OFF + __uint_as_float(zn[rt][u]));
      }
    }
    issue_w(it + 1 < nit);
    // (SAME: a block that is not there has step sizes and activations of zero)
    if (SAME || bc + KSTEP * kw < nblk) {
      const char* xrow = xb + size_t(buf) * TM * 512 + kw * 256;
      const float* xsr = xsb + (buf * 2 + kw) * SUB * TM;
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
        const bool mine = SUB == 1 || f / (4 / SUB) == u;
        f32x4_t acc[2][NTB], xs[NTB];
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) acc[0][tb] = acc[1][tb] = xs[tb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const bf16x8_t q0 = code_frag<BITS>(R[0], m, cm), q1 = code_frag<BITS>(R[1], m, cm);
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb) {
            uint4 v = *reinterpret_cast<const uint4*>(xrow + (16 * tb + i) * 512 + 16 * ((4 * f + m) ^ i));
            if constexpr (SUB > 1)
              v = make_uint4(mine ? v.x : 0u, mine ? v.y : 0u, mine ? v.z : 0u, mine ? v.w : 0u);
            const bf16x8_t xv = __builtin_bit_cast(bf16x8_t, v);
            acc[0][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv, q0, acc[0][tb], 0, 0, 0);
            acc[1][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv, q1, acc[1][tb], 0, 0, 0);
            if constexpr (SAME) xs[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv, ones, xs[tb], 0, 0, 0);
          }
        }
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) {
          if constexpr (!SAME) xs[tb] = *reinterpret_cast<const f32x4_t*>(xsr + u * TM + 16 * tb + 4 * f);
#pragma unroll
          for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              y[rt][tb][r] = __builtin_fmaf(hh[rt][u], __builtin_fmaf(nz[rt][u], xs[tb][r], acc[rt][tb][r]),
                                            y[rt][tb][r]);
        }
      }
    }
    if (next(bc)) end_share();
    stage(buf ^ 1);
    issue_x(it + 2 < nit);
    lds_barrier();
  }
  if (!SAME) end_share();

  // the second K half's sums through LDS, added to the first's
  float* red = reinterpret_cast<float*>(lds_q);   // [4 waves][2][TM][PITCH]
  if (kw == 1) {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          red[((wn * 2 + rt) * TM + 16 * tb + 4 * f + r) * PM_RED_PITCH + i] = total[rt][tb][r];
  }
  __syncthreads();
  if (kw == 0) {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const int64_t o = o0 + 16 * rt + i;
      const float bb = bias && o < c_out ? bias[o] : 0.f;
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int t = 16 * tb + 4 * f + r;
          const float v = total[rt][tb][r] + red[((wn * 2 + rt) * TM + t) * PM_RED_PITCH + i] + bb;
          if (t0 + t < n_tok && o < c_out) {
            const int64_t at = int64_t(t0 + t) * c_out + o;
            if (y_bf16) static_cast<uint16_t*>(Y)[at] = f2bf(v);
            else static_cast<float*>(Y)[at] = v;
          }
        }
    }
  }
}

// Lets the kernel take up to PL_LDS_MAX bytes of dynamic LDS on the current
// device and tells how many workgroups of it with `lds` bytes each the device
// keeps resident (cached per kernel, LDS size and device).
hipError_t resident(const void* kernel, int threads, size_t lds, int* n) {
  struct Entry { const void* k; size_t lds; int dev, n; };
  static std::mutex mu;
  static std::vector<Entry> cache;
  int dev = 0, cus = 0, per = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> g(mu);
  for (const Entry& c : cache)
    if (c.k == kernel && c.lds == lds && c.dev == dev) {
      *n = c.n;
      return hipSuccess;
    }
  if ((e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, int(PL_LDS_MAX))) != hipSuccess ||
      (e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess ||
      (e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, lds)) != hipSuccess)
    return e;
  *n = std::max(1, cus * per);
  cache.push_back(Entry{kernel, lds, dev, *n});
  return hipSuccess;
}

template <int BITS, int TT, int RT, int SUB, int D, bool A16>
hipError_t launch_mfma(const LinArgs& a, const uint16_t* X, int n_tok, void* Y) {
  auto k = packed_mfma_kernel<BITS, TT, RT, SUB, D, A16>;
  const size_t lds = MfmaCfg<BITS, TT, RT, SUB>::lds(D, a.c_in, n_tok, a.bias != nullptr);
  int n = 0;
  const hipError_t e = resident(reinterpret_cast<const void*>(k), PM_THREADS, lds, &n);
  if (e != hipSuccess) return e;
  const int64_t ntile = (a.c_out + 16 * RT - 1) / (16 * RT);
  if (a.bias) n = int(std::max<int64_t>(n, (ntile + PM_BIAS_TILES - 1) / PM_BIAS_TILES));
  hipLaunchKernelGGL(k, dim3(unsigned(std::min<int64_t>(ntile, n))), dim3(PM_THREADS), lds, a.stream, X, n_tok,
                     a.c_in, a.packed, a.ng, a.group_inv, a.h, a.z, a.bias, a.c_out, Y, a.y_bf16, int(ntile));
  return hipGetLastError();
}

// Two row tiles per workgroup share a block's activations and their sums (4096
// channels, W3 g128, one token, 22016 rows: 16.4 -> 13.9 us), but halve the
// workgroups: from 16384 rows, or from 12288 where more than 8 tokens make the
// activations dearer (12 tokens: 12.9 -> 12.3 us), or 4096 where two parts per
// block double that work (W2 g64, 4 tokens, 5120 rows: 11.1 -> 9.7 us); fewer
// rows measured slower (4096 rows, g128, one token: 6.0 -> 7.2 us).  One token
// leaves little to share and takes one tile (44032 x 8192: W4 46.6 -> 42.1 us, W6 67.7
// -> 59.2, W2 35.5 -> 33.2), except at 3 bits (42.7 with two, 44.5 with one) and at
// most 4096 channels of up to 4 bits (22016 x 4096, W4: 14.6 with two, 14.9 with one).
// 5 to 8 tokens have rings of their own (12288 x 4096, W4, 8 tokens: 14.3 us in rings
// of 16 tokens, 11.7 in rings of 8; two tiles 13.1; 13824 x 5120: one 17.8, two 16.4).
// The rings are two units deep: deeper ones cost
// more in resident workgroups than they hide (four: 40.1 -> 44.7 us over a 7B block's linears).
template <int BITS, int TT, int SUB>
hipError_t launch_mfma_rt(const LinArgs& a, const uint16_t* X, int n_tok, void* Y) {
  // rows that are no whole 16-byte chunks (never with whole blocks): dword copies
  if constexpr (SUB > 1) {
    if (a.c_in % PM_BLOCK) return launch_mfma<BITS, TT, 1, SUB, 2, false>(a, X, n_tok, Y);
  }
  if constexpr (TT < 32 && MfmaCfg<BITS, TT, 2, SUB>::FITS) {
    const bool one = TT == 4 && SUB == 1 && n_tok == 1 && (BITS >= 5 || (BITS != 3 && a.c_in > 4096));
    const int64_t from = SUB == 2 ? 4096 : TT == 4 ? 16384 : TT == 8 ? 13312 : TT == 16 ? 12288 : 8192;
    if (!one && a.c_out >= from && MfmaCfg<BITS, TT, 2, SUB>::lds(2, a.c_in, n_tok, a.bias != nullptr) <= PL_LDS_MAX)
      return launch_mfma<BITS, TT, 2, SUB, 2, true>(a, X, n_tok, Y);
  }
  return launch_mfma<BITS, TT, 1, SUB, 2, true>(a, X, n_tok, Y);
}

template <int BITS, int RT>
hipError_t launch_wide(const LinArgs& a, const uint16_t* X, int n_tok, void* Y) {
  auto k = packed_wide_kernel<BITS, RT>;
  constexpr size_t lds = size_t(PM_WAVES) * 2 * PW_TOKENS * 256;
  static_assert(lds >= size_t(PM_WAVES) * RT * PW_TOKENS * PM_RED_PITCH * 4, "partial outputs");
  int n = 0;
  const hipError_t e = resident(reinterpret_cast<const void*>(k), PM_THREADS, lds, &n);   // (allows the LDS)
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(unsigned((a.c_out + 16 * RT - 1) / (16 * RT))), dim3(PM_THREADS), lds, a.stream, X,
                     n_tok, a.c_in, a.packed, a.ng, a.group_inv, a.h, a.z, a.bias, a.c_out, Y, a.y_bf16);
  return hipGetLastError();
}

// 25 to 32 tokens in groups of whole blocks: whether two row tiles per workgroup
// pay.  One workgroup with 32 tokens' activations fits a compute unit, so 256 run
// at a time, and two tiles take about 7/4 of a ring workgroup's time (3/2 of one's
// through registers, the only way with 6 and 7 bits): 8192 rows of 8192 channels
// are one round of the two-tile kernel instead of two (W4, 32 tokens: 25.0 -> 21.5
// us; 22016 x 4096: 38.7 -> 31.7), 12288 rows two instead of three (W2 x 4096: 17.3
// -> 19.3), 4096 rows one as well (W4 x 11008: 18 -> 24.6).
int64_t rounds_of(int64_t c_out, int rows) { return ((c_out + rows - 1) / rows + 255) / 256; }
template <int BITS>
bool two_tiles(int64_t c_out) {
  const int64_t two = rounds_of(c_out, 32), one = rounds_of(c_out, 16);
  return BITS >= 6 ? 3 * two < 2 * one : 7 * two < 4 * one;
}

template <int BITS, int NTB, int SUB>
hipError_t launch_tile(const LinArgs& a, const uint16_t* X, int64_t n_tok, void* Y) {
  auto k = packed_tile_kernel<BITS, NTB, SUB>;
  constexpr size_t lds = tile_lds<NTB, SUB>();
  int n = 0;
  const hipError_t e = resident(reinterpret_cast<const void*>(k), PM_THREADS, lds, &n);
  if (e != hipSuccess) return e;
  // launches of up to 2^16 tokens (32-bit token counts and block indices)
  for (int64_t t0 = 0; t0 < n_tok; t0 += 65536) {
    const int take = int(std::min<int64_t>(n_tok - t0, 65536));
    const int ntt = (take + 16 * NTB - 1) / (16 * NTB);
    const int64_t blocks = ((a.c_out + PT_N - 1) / PT_N) * ntt;
    void* y = static_cast<char*>(Y) + size_t(t0) * size_t(a.c_out) * (a.y_bf16 ? 2 : 4);
    hipLaunchKernelGGL(k, dim3(unsigned(blocks)), dim3(PM_THREADS), lds, a.stream, X + t0 * a.c_in, take,
                       a.c_in, a.packed, a.ng, a.group_inv, a.h, a.z, a.bias, a.c_out, y, a.y_bf16, ntt);
    const hipError_t l = hipGetLastError();
    if (l != hipSuccess) return l;
  }
  return hipSuccess;
}

size_t vector_lds(int nt, int64_t c_in) { return size_t(nt) * size_t(c_in / 32) * (64 + 4); }

template <int BITS, int NT>
hipError_t launch_vector(const LinArgs& a, const uint16_t* X, int n_tok, void* Y) {
  auto k = packed_linear_kernel<BITS, NT>;
  const size_t lds = vector_lds(NT, a.c_in);
  int n = 0;
  const hipError_t e = resident(reinterpret_cast<const void*>(k), PL_THREADS, lds, &n);
  if (e != hipSuccess) return e;
  const int64_t want = (a.c_out + PL_WAVES * PL_ROWS - 1) / (PL_WAVES * PL_ROWS);
  const int rpg = int(a.c_in / 32 / a.ng);
  const int shift = (rpg & (rpg - 1)) == 0 ? __builtin_ctz(unsigned(rpg)) : -1;
  hipLaunchKernelGGL(k, dim3(unsigned(std::min<int64_t>(want, n))), dim3(PL_THREADS), lds, a.stream, X, n_tok,
                     a.c_in, a.packed, rpg, shift, a.h, a.z, a.bias, a.c_out, Y, a.y_bf16);
  return hipGetLastError();
}

// Prompts of more than 96 tokens take the tiled kernel: its time hardly grows
// until its tiles fill the chip, while the small-batch kernel pays one pass over
// the codes per 32 tokens (a 7B block's linears as one graph, W3 g128: 96 tokens
// 215 us in launches of 32, 97 and 128 tokens 224 us tiled; 500 tokens W4, one by
// one: 1272 us in launches, 450 us tiled).
constexpr int64_t TILE_TOKENS = 97;

template <int BITS, int SUB>
hipError_t linear_sub(const LinArgs& a, const uint16_t* X, int64_t n_tok, void* Y) {
  const size_t es = a.y_bf16 ? 2 : 4;
  if (n_tok >= TILE_TOKENS) return launch_tile<BITS, 4, SUB>(a, X, n_tok, Y);
  const bool bias = a.bias != nullptr;
  if (SUB > 1 && n_tok <= 2 && vector_lds(int(n_tok), a.c_in) <= PL_LDS_MAX)
    return n_tok == 1 ? launch_vector<BITS, 1>(a, X, 1, Y) : launch_vector<BITS, 2>(a, X, 2, Y);
  for (int64_t t0 = 0; t0 < n_tok;) {
    int take = int(std::min<int64_t>(n_tok - t0, 32));
    // 33 to 48 tokens at 6 and 7 bits where two row tiles save few rounds: 24 and the
    // rest (27648 x 5120, 48 tokens: 96 us, 105 as 32 and 16; 24576 x 8192: 130 and 115)
    if (SUB == 1 && BITS >= 6 && n_tok - t0 > 32 && n_tok - t0 <= 48 &&
        9 * rounds_of(a.c_out, 32) > 5 * rounds_of(a.c_out, 16))
      take = 24;
    // 32 tokens where their rings fit LDS (not with wide codes), else 24
    constexpr bool T32 = MfmaCfg<BITS, 32, 1, SUB>::FITS && !(SUB == 1 && BITS >= 6);
    // (through registers also where codes are too wide for rings of 32: 6 and 7 bits, 32 tokens, 4096 x 4096
    // 13.4 us in launches of 24 and 8, 9.0 in one)
    const bool two = two_tiles<BITS>(a.c_out), wide = SUB == 1 && take > 24 && (BITS >= 6 || two);
    if (!wide && take > 24 && (!T32 || MfmaCfg<BITS, 32, 1, SUB>::lds(2, a.c_in, take, bias) > PL_LDS_MAX)) take = 24;
    const uint16_t* x = X + t0 * a.c_in;
    void* y = static_cast<char*>(Y) + size_t(t0) * size_t(a.c_out) * es;
    // up to 4 tokens are kept in LDS where they fit
    const bool keep = take <= 4 && MfmaCfg<BITS, 4, 1, SUB>::lds(2, a.c_in, take, bias) <= PL_LDS_MAX;
    const hipError_t e = keep         ? launch_mfma_rt<BITS, 4, SUB>(a, x, take, y)
                         : wide       ? (BITS >= 6 && !two ? launch_wide<BITS, 1>(a, x, take, y) : launch_wide<BITS, 2>(a, x, take, y))
                         : take <= 8  ? launch_mfma_rt<BITS, 8, SUB>(a, x, take, y)
                         : take <= 16 ? launch_mfma_rt<BITS, 16, SUB>(a, x, take, y)
                         : take <= 24 ? launch_mfma_rt<BITS, 24, SUB>(a, x, take, y)
                                      : launch_mfma_rt<BITS, T32 ? 32 : 24, SUB>(a, x, take, y);
    if (e != hipSuccess) return e;
    t0 += take;
  }
  return hipSuccess;
}

}  // namespace

template <int BITS>
hipError_t linear_bits(const LinArgs& a, int64_t group, const uint16_t* X, int64_t n_tok, void* Y) {
  if (group % 128 == 0) return linear_sub<BITS, 1>(a, X, n_tok, Y);
  if (group % 64 == 0) return linear_sub<BITS, 2>(a, X, n_tok, Y);
  return linear_sub<BITS, 4>(a, X, n_tok, Y);
}

}  // namespace oq
