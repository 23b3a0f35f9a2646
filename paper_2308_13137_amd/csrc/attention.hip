// Causal multi-head attention for the whole-block calibration step (the
// attention operation of Sec. 3.3 with the quantised Q^, K^, V^ of Eq. 5),
// forward and backward, on bf16 matrix cores (v_mfma_f32_16x16x32_bf16).
//
// Layouts: Q^ [T, H d], K^ and V^ [T, Hkv d] bf16, token-major with the
// heads side by side (T = n_seq * S, the samples one after another); query
// head h reads key/value head h / (H / Hkv).  O and the gradients fp32 in
// the same layouts; the per-query softmax statistic LSE [H, T] is kept in
// base 2 of the scaled logits (t = s * log2(e) / sqrt(d)).
//
// Forward (one workgroup = 64 queries of one head, four waves of 16): each
// wave computes S^T = K Q^T for a 64-key tile (keys on the matrix rows), so
// a lane's accumulators all belong to one query: the online softmax needs
// only in-lane work and two cross-lane exchanges, and the probabilities feed
// the O^T = V^T P product as its B operand straight from registers (the
// k-order of the product is permuted to match: any consistent order of the
// summed index gives the same sum).  K is staged in LDS row-major (XOR
// swizzled chunks), V transposed (padded rows).
//
// Backward (deterministic, no atomics): one kernel per 64-query tile forms
// D = sum_j P_ij dP_ij in a first sweep over the key tiles (written out for
// the other kernel, which runs after it) and accumulates dQ in a second; one
// kernel per 64-key tile and key head accumulates dK, dV over every query tile
// and query head of its group.  S and dP are recomputed from LSE in the
// orientation whose accumulators are the next product's operand as they stand.
//
// Rounding: P and dS enter the matrix cores as bf16.  Block inputs share
// outlier channels, so Q^, K^, V^ rows carry a large component common to all
// tokens; two exact identities cancel it (the weights of a softmax row sum to
// one, a row of dS sums to zero) and the kernels keep both under rounding: O
// is divided by the sum of the bf16 weights that entered its product, and dS
// enters the dQ and dK products as a hi + lo pair of bf16 terms.  The online
// maximum is kept integral (a power-of-two rescaling is exact), so the bf16
// weights of a row are bf16(2^(t - ceil(max t))) up to one common power of
// two, independent of the order of the key tiles.
#include <math.h>

#include "common.h"
#include "oq_internal.h"

namespace oq {
namespace {

constexpr int AT = 64;          // queries / keys per tile
constexpr int ANT = 256;        // threads per workgroup (4 waves)

typedef uint16_t bf16raw;

OQ_DEV bf16x8_t bits_as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8_t, v); }
OQ_DEV f32x4_t mfma(bf16x8_t a, bf16x8_t b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
OQ_DEV uint32_t pack2(float a, float b) { return f2bf2(a, b); }

// The query tile (of nt per sample), head and sample of a workgroup: heads
// vary fastest, so consecutive workgroups, which go to different XCDs, have
// equal lengths and an XCD sees all tiles of its heads (their K and V stay in
// its L2); the longest tiles come first.  With the tile index fastest and a
// tile count that is a multiple of eight, XCD k would get tiles k, k + 8, ...
// of every head: up to 1.4 times the average work (2048 tokens, 128-query
// tiles).
struct AttnTile {
  int qt, h, b;
};
OQ_DEV AttnTile attn_tile(int H, int n_seq, int nt) {
  const int x = int(blockIdx.x), r = x / H;
  return {nt - 1 - r / n_seq, x % H, r % n_seq};
}

// Row-major [64][DH] bf16 tile ("K layout"), 16-byte chunk c of row r at
// slot c ^ (r & (NCH-1)).
template <int DH>
OQ_DEV bf16x8_t read_rm(const uint4* lds, int r, int c) {
  constexpr int NCH = DH / 8;
  return bits_as_bf16x8(lds[r * NCH + (c ^ (r & (NCH - 1)))]);
}

// ------------------------------------------------------------------ forward
// Row-major [64][DH] bf16 tile in 32-byte blocks, block b of row r at
// b ^ vswz(r): the four rows one transposed read of a 16-lane group touches
// (and the next group's four) fall in distinct banks.
template <int DH>
OQ_DEV int vswz(int r) {
  return (r + 4 * (r >> 3)) & (DH / 16 - 1);
}
// Global -> registers: this thread's chunks of a 64-row tile (NCH 16-byte
// chunks per row), chunk idx = tid + ANT * i.
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
template <int DH>
OQ_DEV void tile_to_regs(u32x4_t (&v)[AT * DH / 8 / ANT], const bf16raw* g, int64_t ld, int tid) {
  constexpr int NCH = DH / 8;
#pragma unroll
  for (int i = 0; i < AT * NCH / ANT; ++i) {
    const int idx = tid + ANT * i;
    v[i] = *reinterpret_cast<const u32x4_t*>(g + (idx / NCH) * ld + 8 * (idx % NCH));
  }
}
// registers -> LDS, K layout (16-byte chunk c of row r at c ^ (r & (NCH-1)))
template <int DH>
OQ_DEV void regs_to_k(uint4* lds, const u32x4_t (&v)[AT * DH / 8 / ANT], int tid) {
  constexpr int NCH = DH / 8;
#pragma unroll
  for (int i = 0; i < AT * NCH / ANT; ++i) {
    const int idx = tid + ANT * i;
    const int r = idx / NCH, c = idx % NCH;
    reinterpret_cast<u32x4_t*>(lds)[r * NCH + (c ^ (r & (NCH - 1)))] = v[i];
  }
}
// registers -> LDS, V layout (32-byte block b of row r at b ^ vswz(r))
template <int DH>
OQ_DEV void regs_to_v(uint4* lds, const u32x4_t (&v)[AT * DH / 8 / ANT], int tid) {
  constexpr int NCH = DH / 8;
#pragma unroll
  for (int i = 0; i < AT * NCH / ANT; ++i) {
    const int idx = tid + ANT * i;
    const int r = idx / NCH, c = idx % NCH;
    reinterpret_cast<u32x4_t*>(lds)[r * NCH + 2 * ((c >> 1) ^ vswz<DH>(r)) + (c & 1)] = v[i];
  }
}
// A operand of O^T = V^T P for rows d = 16 j .. 16 j + 15 and the k-chunk k2,
// in the k order of the P operand: lane (fk, i) needs keys 32 k2 + 4 fk + 0..3
// and 32 k2 + 16 + 4 fk + 0..3 of column d = 16 j + i.  ds_read_b64_tr_b16
// gives lane i of a 16-lane group four consecutive rows k0..k0+3 of column
// 16 j + i when lane j' of the group points at row k0 + j'/4, columns
// 16 j + 4 (j' % 4) .. + 3.
template <int DH>
OQ_DEV bf16x8_t v_frag(const uint4* sV, int j, int k2, int lane) {
  typedef short v4i16 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) v4i16 lds_v4;
  const int fk = lane >> 4, jj = lane & 15;
  const int r0 = 32 * k2 + 4 * fk + (jj >> 2), r1 = r0 + 16;
  const char* base = reinterpret_cast<const char*>(sV);
  const char* a0 = base + r0 * (2 * DH) + 32 * (j ^ vswz<DH>(r0)) + 8 * (jj & 3);
  const char* a1 = base + r1 * (2 * DH) + 32 * (j ^ vswz<DH>(r1)) + 8 * (jj & 3);
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(a0));
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(a1));
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int DH>
__global__ __launch_bounds__(ANT) void attn_fwd_kernel(const bf16raw* __restrict__ Q,
                                                       const bf16raw* __restrict__ K,
                                                       const bf16raw* __restrict__ V, int S,
                                                       int H, int Hkv, float* __restrict__ O,
                                                       float* __restrict__ LSE, int64_t T) {
  constexpr int KS = DH / 32;        // k-steps of the S product
  constexpr int JD = DH / 16;        // 16-row tiles of O^T
  constexpr int NR = AT * DH / 8 / ANT;
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  __shared__ uint4 sK[AT * DH / 8];
  __shared__ uint4 sV[AT * DH / 8];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int fr = lane & 15, fk = lane >> 4;
  const AttnTile at = attn_tile(H, int(T / S), S / AT);
  const int qt = at.qt, h = at.h, b = at.b;
  const int g = h / (H / Hkv);
  const int64_t ldq = int64_t(H) * DH, ldk = int64_t(Hkv) * DH;
  const int64_t row0 = int64_t(b) * S;
  const int qrow = qt * AT + 16 * wave + fr;            // this lane's query within the sample
  const float sc = 1.4426950408889634f / sqrtf(float(DH));
  const bf16x2_t ones = {(__bf16)1.0f, (__bf16)1.0f};

  bf16x8_t qf[KS];
  {
    const bf16raw* qp = Q + (row0 + qrow) * ldq + int64_t(h) * DH;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[ks] = bits_as_bf16x8(*reinterpret_cast<const uint4*>(qp + 32 * ks + 8 * fk));
  }
  f32x4_t acc[JD];
#pragma unroll
  for (int j = 0; j < JD; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f, l_b = 0.f;
  u32x4_t kr[NR], vr[NR];
  tile_to_regs<DH>(kr, K + row0 * ldk + int64_t(g) * DH, ldk, tid);
  tile_to_regs<DH>(vr, V + row0 * ldk + int64_t(g) * DH, ldk, tid);

  for (int kt = 0; kt <= qt; ++kt) {
    __syncthreads();
    regs_to_k<DH>(sK, kr, tid);
    regs_to_v<DH>(sV, vr, tid);
    __syncthreads();
    {                                                    // the next tile, in flight meanwhile
      const int64_t krow = row0 + int64_t(kt < qt ? kt + 1 : kt) * AT;
      tile_to_regs<DH>(kr, K + krow * ldk + int64_t(g) * DH, ldk, tid);
      tile_to_regs<DH>(vr, V + krow * ldk + int64_t(g) * DH, ldk, tid);
    }
    // S^T [64 keys x 16 queries of this wave]: lane holds key 16 i + 4 fk + r, query fr
    f32x4_t st[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      st[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        st[i] = mfma(read_rm<DH>(sK, 16 * i + fr, 4 * ks + fk), qf[ks], st[i]);
    }
    if (kt == qt) {                                      // the diagonal tile: causal mask
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (kt * AT + 16 * i + 4 * fk + r > qrow) st[i][r] = -INFINITY;
    }
    float mt = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) mt = fmaxf(fmaxf(mt, fmaxf(st[i][0], st[i][1])), fmaxf(st[i][2], st[i][3]));
    mt = fmaxf(mt, __shfl_xor(mt, 16));
    mt = fmaxf(mt, __shfl_xor(mt, 32));
    // the running maximum stays an integer, so every rescaling is an exact
    // power of two: each weight reaching the PV product is bf16(2^(t - M))
    // times a power of two, M the row's final maximum, whatever the tile order
    const float mn = fmaxf(m, ceilf(mt * sc));
    float ls = 0.f, lr = 0.f;
    bf16x8_t pb[2];
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 2 * k2 + (e >> 1), r0 = 2 * (e & 1);
        const float p0 = __builtin_amdgcn_exp2f(fmaf(st[i][r0], sc, -mn));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(st[i][r0 + 1], sc, -mn));
        ls += p0 + p1;
        w[e] = pack2(p0, p1);
        // the weights the PV product sees are these bf16 values: their own
        // sum normalises O (an exact weighted mean of V rows); l (unrounded)
        // gives LSE
        lr = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w[e]), ones, lr, false);
      }
      pb[k2] = bits_as_bf16x8(make_uint4(w[0], w[1], w[2], w[3]));
    }
    ls += __shfl_xor(ls, 16);
    ls += __shfl_xor(ls, 32);
    lr += __shfl_xor(lr, 16);
    lr += __shfl_xor(lr, 32);
    if (__any(mn != m)) {
      const float alpha = m == -INFINITY ? 0.0f : ldexpf(1.0f, int(m - mn));
      l *= alpha;
      l_b *= alpha;
#pragma unroll
      for (int j = 0; j < JD; ++j) acc[j] = acc[j] * alpha;
    }
    l += ls;
    l_b += lr;
    m = mn;
#pragma unroll
    for (int j = 0; j < JD; ++j)
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) acc[j] = mfma(v_frag<DH>(sV, j, k2, lane), pb[k2], acc[j]);
  }
  const float inv = 1.0f / l_b;
  float* op = O + (row0 + qrow) * ldq + int64_t(h) * DH;
#pragma unroll
  for (int j = 0; j < JD; ++j)
    *reinterpret_cast<float4*>(op + 16 * j + 4 * fk) =
        make_float4(acc[j][0] * inv, acc[j][1] * inv, acc[j][2] * inv, acc[j][3] * inv);
  if (fk == 0) LSE[int64_t(h) * T + row0 + qrow] = m + log2f(l);
}

// The same forward with 32 queries per wave (128 per workgroup, S a multiple
// of 128): every K and V fragment read from LDS feeds two matrix
// instructions, one per 16-query half, which halves the LDS traffic per
// instruction.  Arithmetic per query is the kernel's above, unchanged.
template <int DH>
__global__ __launch_bounds__(ANT) void attn_fwd2_kernel(const bf16raw* __restrict__ Q,
                                                        const bf16raw* __restrict__ K,
                                                        const bf16raw* __restrict__ V, int S,
                                                        int H, int Hkv, float* __restrict__ O,
                                                        float* __restrict__ LSE, int64_t T) {
  constexpr int KS = DH / 32;
  constexpr int JD = DH / 16;
  constexpr int NR = AT * DH / 8 / ANT;
  constexpr int QW = 2 * AT;                           // queries per workgroup
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  __shared__ uint4 sK[AT * DH / 8];
  __shared__ uint4 sV[AT * DH / 8];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int fr = lane & 15, fk = lane >> 4;
  const AttnTile at = attn_tile(H, int(T / S), S / QW);
  const int qt = at.qt, h = at.h, b = at.b;
  const int g = h / (H / Hkv);
  const int64_t ldq = int64_t(H) * DH, ldk = int64_t(Hkv) * DH;
  const int64_t row0 = int64_t(b) * S;
  int qrow[2];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) qrow[hh] = qt * QW + 32 * wave + 16 * hh + fr;
  const float sc = 1.4426950408889634f / sqrtf(float(DH));
  const bf16x2_t ones = {(__bf16)1.0f, (__bf16)1.0f};

  bf16x8_t qf[2][KS];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const bf16raw* qp = Q + (row0 + qrow[hh]) * ldq + int64_t(h) * DH;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[hh][ks] = bits_as_bf16x8(*reinterpret_cast<const uint4*>(qp + 32 * ks + 8 * fk));
  }
  f32x4_t acc[2][JD];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int j = 0; j < JD; ++j) acc[hh][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f}, l_b[2] = {0.f, 0.f};
  u32x4_t kr[NR], vr[NR];
  tile_to_regs<DH>(kr, K + row0 * ldk + int64_t(g) * DH, ldk, tid);
  tile_to_regs<DH>(vr, V + row0 * ldk + int64_t(g) * DH, ldk, tid);
  const int nk = 2 * qt + 2;                           // key tiles up to the diagonal
  for (int kt = 0; kt < nk; ++kt) {
    __syncthreads();
    regs_to_k<DH>(sK, kr, tid);
    regs_to_v<DH>(sV, vr, tid);
    __syncthreads();
    {
      const int64_t krow = row0 + int64_t(kt + 1 < nk ? kt + 1 : kt) * AT;
      tile_to_regs<DH>(kr, K + krow * ldk + int64_t(g) * DH, ldk, tid);
      tile_to_regs<DH>(vr, V + krow * ldk + int64_t(g) * DH, ldk, tid);
    }
    // S^T [64 keys x 16 queries] per half: lane holds key 16 i + 4 fk + r, query fr
    f32x4_t st[2][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      st[0][i] = st[1][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8_t kf = read_rm<DH>(sK, 16 * i + fr, 4 * ks + fk);
        st[0][i] = mfma(kf, qf[0][ks], st[0][i]);
        st[1][i] = mfma(kf, qf[1][ks], st[1][i]);
      }
    }
    if (kt >= 2 * qt) {                                // the tiles the diagonal crosses
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (kt * AT + 16 * i + 4 * fk + r > qrow[hh]) st[hh][i][r] = -INFINITY;
    }
    bf16x8_t pb[2][2];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      float mt = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        mt = fmaxf(fmaxf(mt, fmaxf(st[hh][i][0], st[hh][i][1])), fmaxf(st[hh][i][2], st[hh][i][3]));
      mt = fmaxf(mt, __shfl_xor(mt, 16));
      mt = fmaxf(mt, __shfl_xor(mt, 32));
      const float mn = fmaxf(m[hh], ceilf(mt * sc));
      float ls = 0.f, lr = 0.f;
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) {
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 2 * k2 + (e >> 1), r0 = 2 * (e & 1);
          const float p0 = __builtin_amdgcn_exp2f(fmaf(st[hh][i][r0], sc, -mn));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(st[hh][i][r0 + 1], sc, -mn));
          ls += p0 + p1;
          w[e] = pack2(p0, p1);
          lr = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w[e]), ones, lr, false);
        }
        pb[hh][k2] = bits_as_bf16x8(make_uint4(w[0], w[1], w[2], w[3]));
      }
      ls += __shfl_xor(ls, 16);
      ls += __shfl_xor(ls, 32);
      lr += __shfl_xor(lr, 16);
      lr += __shfl_xor(lr, 32);
      if (__any(mn != m[hh])) {
        // a row whose first tile is wholly masked keeps m = -inf until its
        // first key arrives: alpha 0 leaves its (zero) sums as they are
        const float alpha = m[hh] == -INFINITY ? 0.0f : ldexpf(1.0f, int(m[hh] - mn));
        l[hh] *= alpha;
        l_b[hh] *= alpha;
#pragma unroll
        for (int j = 0; j < JD; ++j) acc[hh][j] = acc[hh][j] * alpha;
      }
      l[hh] += ls;
      l_b[hh] += lr;
      m[hh] = mn;
    }
#pragma unroll
    for (int j = 0; j < JD; ++j)
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) {
        const bf16x8_t vf = v_frag<DH>(sV, j, k2, lane);
        acc[0][j] = mfma(vf, pb[0][k2], acc[0][j]);
        acc[1][j] = mfma(vf, pb[1][k2], acc[1][j]);
      }
  }
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const float inv = 1.0f / l_b[hh];
    float* op = O + (row0 + qrow[hh]) * ldq + int64_t(h) * DH;
#pragma unroll
    for (int j = 0; j < JD; ++j)
      *reinterpret_cast<float4*>(op + 16 * j + 4 * fk) =
          make_float4(acc[hh][j][0] * inv, acc[hh][j][1] * inv, acc[hh][j][2] * inv,
                      acc[hh][j][3] * inv);
    if (fk == 0) LSE[int64_t(h) * T + row0 + qrow[hh]] = m[hh] + log2f(l[hh]);
  }
}

// ------------------------------------------------------------------ forward, quantised softmax
// The ablation on softmax quantisation: every query row of probabilities
// goes through Q_a (per-row asymmetric MinMax, the activation quantiser's
// fp32 order) before the product with V.  A row's range must be known before
// any of its values is quantised, so the kernel sweeps the key tiles twice:
// the first forms LSE (integral running maximum, as the forward above) and
// the extreme logits, the second recomputes P = 2^(t - LSE), quantises it
// with the row's (max, min) and accumulates O = sum P^ V (no renormalisation:
// P^ approximates the normalised row).  Row record pstat [H, T, 4]:
// (max P, min P, lowest index holding each) -- the masked entries of a row
// are zeros, so every row but a sample's last has min 0.
template <int DH>
__global__ __launch_bounds__(ANT) void attn_fwd_q_kernel(const bf16raw* __restrict__ Q,
                                                         const bf16raw* __restrict__ K,
                                                         const bf16raw* __restrict__ V, int S,
                                                         int H, int Hkv, int p_bits,
                                                         float* __restrict__ O,
                                                         float* __restrict__ LSE,
                                                         float4* __restrict__ pstat, int64_t T) {
  constexpr int KS = DH / 32, JD = DH / 16, NR = AT * DH / 8 / ANT;
  __shared__ uint4 sK[AT * DH / 8];
  __shared__ uint4 sV[AT * DH / 8];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int fr = lane & 15, fk = lane >> 4;
  const int ntile = S / AT;
  const AttnTile at = attn_tile(H, int(T / S), ntile);
  const int qt = at.qt, h = at.h, b = at.b;
  const int g = h / (H / Hkv);
  const int64_t ldq = int64_t(H) * DH, ldk = int64_t(Hkv) * DH;
  const int64_t row0 = int64_t(b) * S;
  const int qrow = qt * AT + 16 * wave + fr;
  const float sc = 1.4426950408889634f / sqrtf(float(DH));
  const float qmax = float((1 << p_bits) - 1);

  bf16x8_t qf[KS];
  {
    const bf16raw* qp = Q + (row0 + qrow) * ldq + int64_t(h) * DH;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[ks] = bits_as_bf16x8(*reinterpret_cast<const uint4*>(qp + 32 * ks + 8 * fk));
  }
  f32x4_t acc[JD];
#pragma unroll
  for (int j = 0; j < JD; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f, smax = -INFINITY, smin = INFINITY, lse = 0.f;
  QParams prm{};
  float pmx = 0.f, pmn = 0.f;
  int amax = INT_MAX, amin = INT_MAX;
  u32x4_t kr[NR], vr[NR];
  const int nk = qt + 1;
  auto fetch = [&](int t) {
    const int64_t krow = row0 + int64_t(t) * AT;
    tile_to_regs<DH>(kr, K + krow * ldk + int64_t(g) * DH, ldk, tid);
    tile_to_regs<DH>(vr, V + krow * ldk + int64_t(g) * DH, ldk, tid);
  };
  fetch(0);
  for (int it = 0; it < 2 * nk; ++it) {
    const int kt = it < nk ? it : it - nk;
    __syncthreads();
    regs_to_k<DH>(sK, kr, tid);
    regs_to_v<DH>(sV, vr, tid);
    __syncthreads();
    fetch(kt + 1 < nk ? kt + 1 : 0);
    f32x4_t st[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      st[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        st[i] = mfma(read_rm<DH>(sK, 16 * i + fr, 4 * ks + fk), qf[ks], st[i]);
    }
    if (kt == qt) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (kt * AT + 16 * i + 4 * fk + r > qrow) st[i][r] = -INFINITY;
    }
    if (it < nk) {
      // sweep 1: LSE as the forward forms it, and the row's extreme logits
      float mt = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          mt = fmaxf(mt, st[i][r]);
          if (st[i][r] != -INFINITY) smin = fminf(smin, st[i][r]);
        }
      smax = fmaxf(smax, mt);
      mt = fmaxf(mt, __shfl_xor(mt, 16));
      mt = fmaxf(mt, __shfl_xor(mt, 32));
      const float mn_ = fmaxf(m, ceilf(mt * sc));
      float ls = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) ls += __builtin_amdgcn_exp2f(fmaf(st[i][r], sc, -mn_));
      ls += __shfl_xor(ls, 16);
      ls += __shfl_xor(ls, 32);
      l = (m == -INFINITY ? 0.0f : l * ldexpf(1.0f, int(m - mn_))) + ls;
      m = mn_;
      if (it == nk - 1) {
        smax = fmaxf(smax, __shfl_xor(smax, 16));
        smax = fmaxf(smax, __shfl_xor(smax, 32));
        smin = fminf(smin, __shfl_xor(smin, 16));
        smin = fminf(smin, __shfl_xor(smin, 32));
        lse = m + log2f(l);
        // the row's extreme probabilities, computed as each element's is
        pmx = __builtin_amdgcn_exp2f(fmaf(smax, sc, -lse));
        pmn = qrow < S - 1 ? 0.0f : __builtin_amdgcn_exp2f(fmaf(smin, sc, -lse));
        prm = make_qparams(pmx, pmn, 1.0f, 1.0f, qmax);
      }
      continue;
    }
    // sweep 2: P, its quantisation, and O += P^ V
    bf16x8_t pb[2];
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 2 * k2 + (e >> 1), r0 = 2 * (e & 1);
        float pq[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const float p = __builtin_amdgcn_exp2f(fmaf(st[i][r0 + c], sc, -lse));
          const int key = kt * AT + 16 * i + 4 * fk + r0 + c;
          if (p == pmx) amax = min(amax, key);
          if (p == pmn) amin = min(amin, key);
          pq[c] = dequant(quant_elem(p, prm, qmax).q, prm);
        }
        w[e] = pack2(pq[0], pq[1]);
      }
      pb[k2] = bits_as_bf16x8(make_uint4(w[0], w[1], w[2], w[3]));
    }
#pragma unroll
    for (int j = 0; j < JD; ++j)
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) acc[j] = mfma(v_frag<DH>(sV, j, k2, lane), pb[k2], acc[j]);
  }
  amax = min(amax, __shfl_xor(amax, 16));
  amax = min(amax, __shfl_xor(amax, 32));
  amin = min(amin, __shfl_xor(amin, 16));
  amin = min(amin, __shfl_xor(amin, 32));
  // a masked key past the visited tiles is the first zero if none came before
  if (amin == INT_MAX) amin = qrow + 1;
  float* op = O + (row0 + qrow) * ldq + int64_t(h) * DH;
#pragma unroll
  for (int j = 0; j < JD; ++j)
    *reinterpret_cast<float4*>(op + 16 * j + 4 * fk) =
        make_float4(acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
  if (fk == 0) {
    LSE[int64_t(h) * T + row0 + qrow] = lse;
    pstat[int64_t(h) * T + row0 + qrow] =
        make_float4(pmx, pmn, __int_as_float(amax), __int_as_float(amin));
  }
}

// ------------------------------------------------------------------ backward
// Bound by the exponentials and the vector work around the matrix
// instructions (each about 45% of the time, partly side by side); 32-row
// tiles with more waves per SIMD, 32 rows per wave, and 32-key workgroups were
// no faster.  With P and dS staged through LDS, tiles double buffered in
// registers and the tile index fastest in the grid, the backward of 32 heads
// of 2048 tokens at 128 wide took 498 us, that of 32 heads (four per key head)
// over four samples of 1088 at 64 wide 275; now 209 and 163, the same bits.
// The forwards gained from the grid order alone: 87 -> 68 and 53 -> 44.
// Tiles come from global memory straight into LDS (global_load_lds_dwordx4,
// no registers) and are double buffered: the next tile is in flight while one
// is used, with one barrier per tile.  16-byte chunk c of row r sits at
// c ^ bswz(r).  Three kinds of reads share the layout: an operand's rows in
// the order of row_of or d_row (sixteen rows, one chunk column per 16 lanes)
// and its columns, transposed on the way (ds_read_b64_tr_b16: rows 8 f + 0..3
// or 4..7 for two f, a 32-byte column block each).  bswz puts each on distinct
// banks: of the rows with bit 2 alike, 0-3 and 8-11 take the eight slot pairs,
// 16-19 and 24-27 take them again in the other order and by the other member.
template <int DH>
OQ_DEV int bswz(int r) {
  const int b2 = (r >> 2) & 1, b3 = (r >> 3) & 1, b4 = (r >> 4) & 1;
  return DH == 128 ? ((r & 3) << 1) | ((b3 ^ b4) << 3) | (b4 ^ b2)
                   : (r & 2) | ((b3 ^ b4) << 2) | (b4 ^ b2);
}
template <int DH>
OQ_DEV bf16x8_t row_frag(const uint4* tile, int r, int c) {
  return bits_as_bf16x8(tile[r * (DH / 8) + (c ^ bswz<DH>(r))]);
}
// The row of a 32-row step that row i of its accumulator tile hf stands for: a
// lane's values (rows 4 fk + r of either tile) are then rows 8 fk + 4 hf + r,
// an operand's k order, and feed the next product without leaving the lane.
OQ_DEV int row_of(int hf, int i) { return 8 * (i >> 2) + 4 * hf + (i & 3); }
// The same within 16 rows for the sweep that forms D: blocks of four rows in
// the order 0, 2, 3, 1 (which bswz keeps on distinct banks).
OQ_DEV int d_row(int i) {
  const int b0 = (i >> 2) & 1, b1 = i >> 3;
  return 8 * (b0 ^ b1) + 4 * b1 + (i & 3);
}
// Lane (fk, i) gets rows 32 k2 + 8 fk + 0..7 of column 16 j + i.
template <int DH>
OQ_DEV bf16x8_t col_frag(const uint4* tile, int k2, int j, int lane) {
  typedef short v4i16 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) v4i16 lds_v4;
  const int fk = lane >> 4, jj = lane & 15;
  const int r0 = 8 * fk + (jj >> 2), c = 2 * j + ((jj >> 1) & 1);
  const char* t = reinterpret_cast<const char*>(tile) + 32 * k2 * (2 * DH) + 8 * (jj & 1);
  const char* a0 = t + r0 * (2 * DH) + 16 * (c ^ bswz<DH>(r0));
  const char* a1 = t + (r0 + 4) * (2 * DH) + 16 * (c ^ bswz<DH>(r0) ^ 1);
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(a0));
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(a1));
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// The asynchronous copies are outside the compiler's wait counting: bwd_wait
// stands before the barrier that publishes a tile.
OQ_DEV void bwd_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// A value loaded before a loop, waited for here: left to itself the compiler
// waits at the value's first use inside the loop, where the count would drain
// the copies in flight on every pass.
template <typename V>
OQ_DEV void settle(V& v) {
  asm volatile("" : "+v"(v));
}
typedef int i32x4_t __attribute__((ext_vector_type(4)));
template <typename V, typename E>
OQ_DEV V lds4(const E* p) {
  return *reinterpret_cast<const V*>(p);
}
// four fp32 gradients at any float's address
OQ_DEV void store4(float* p, f32x4_t v) {
  typedef float f32x4u_t __attribute__((ext_vector_type(4), aligned(4)));
  *reinterpret_cast<f32x4u_t*>(p) = v;
}
OQ_DEV bf16x8_t load_frag(const bf16raw* p) {
  return bits_as_bf16x8(*reinterpret_cast<const uint4*>(p));
}
OQ_DEV uint32_t lds_byte(const void* p) {
  return static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void*)(p)));
}
OQ_DEV void dma16(const void* base, uint32_t off, uint32_t lds) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds);
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 2\n\t"
      "global_load_lds_dwordx4 %2, %3\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(m0v), "v"(off), "s"(base)
      : "memory");
}
OQ_DEV void dma4(const void* base, uint32_t off, uint32_t lds) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds);
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 2\n\t"
      "global_load_lds_dword %2, %3\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(m0v), "v"(off), "s"(base)
      : "memory");
}
// A [64][DH] tile at g (row pitch ld): copy i of the workgroup's four waves
// covers rows i * RS .. + RS - 1, lane offsets from tile_off.  bswz has period
// 32; over 16 rows (RS at 128 wide) it flips the slot's bits 0 and 3.
template <int DH>
OQ_DEV uint32_t tile_off(int wave, int lane, int64_t ld) {
  constexpr int NCH = DH / 8;
  const int idx = 64 * wave + lane, r = idx / NCH;
  return uint32_t(r) * uint32_t(2 * ld) + 16u * uint32_t((idx % NCH) ^ bswz<DH>(r));
}
template <int DH>
OQ_DEV void tile_dma(const bf16raw* g, int64_t ld, uint32_t off, uint32_t lds, int wave) {
  constexpr int RS = ANT * 8 / DH;
  static_assert(RS == (DH == 128 ? 16 : 32), "rows per copy");
#pragma unroll
  for (int i = 0; i < AT / RS; ++i)
    dma16(g + int64_t(i * RS) * ld, DH == 128 && (i & 1) ? off ^ (16u * 9u) : off,
          lds + uint32_t((i * 4 + wave) * 1024));
}
// two fp32 values as words of two bf16 operands: hi, and the rounding's remainder lo
OQ_DEV void split2(float a, float b, uint32_t* hi, uint32_t* lo) {
  *hi = pack2(a, b);
  *lo = pack2(a - __uint_as_float(*hi << 16), b - __uint_as_float(*hi & 0xffff0000u));
}

// dK, dV: one workgroup per 64 keys of a key head; each wave owns 16 keys and
// accumulates over every query tile and query head of its group.
// S and dP are recomputed as [queries x keys] tiles (from LSE and D) with the
// queries in the order of row_of: two tiles of a lane's values are the B
// operand (k = queries) of dV^T += dO^T P and dK^T += Q^T dS as they stand.
// QP (softmax quantisation): P^ (the quantised row) enters dV, and dP goes
// through Q_a's straight-through rule: dP = m dP^ plus the routed gradients of
// the row's max and min (from the dQ kernel's first sweep).
template <int DH, bool QP>
__global__ __launch_bounds__(ANT, 2) void attn_bwd_dkv_kernel(
    const bf16raw* __restrict__ Q, const bf16raw* __restrict__ K, const bf16raw* __restrict__ V,
    const bf16raw* __restrict__ dO, const float* __restrict__ LSE, const float* __restrict__ Dl,
    int S, int H, int Hkv, int n_seq, int64_t T, float* __restrict__ dK, float* __restrict__ dV,
    int p_bits, const float4* __restrict__ pstat, const float2* __restrict__ dmm) {
  constexpr int KS = DH / 32, JD = DH / 16;
  constexpr int QB = QP ? AT : 4;
  constexpr int NT = AT * DH / 8;                        // 16-byte chunks of a tile
  __shared__ uint4 sT[2][2 * NT];                       // Q, then dO
  __shared__ __attribute__((aligned(16))) float sL[2][AT], sD[2][AT];
  // QP: per query row h, 1/h, z of Q_a, the routed max / min gradients and
  // the indices that take them
  __shared__ __attribute__((aligned(16))) float sQh[2][QB], sQr[2][QB], sQz[2][QB];
  __shared__ __attribute__((aligned(16))) float sDmx[2][QB], sDmn[2][QB];
  __shared__ __attribute__((aligned(16))) int sAmx[2][QB], sAmn[2][QB];
  const float qmax = QP ? float((1 << p_bits) - 1) : 0.0f;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int fr = lane & 15, fk = lane >> 4;
  int rest = int(blockIdx.x);
  const int g = rest % Hkv;
  rest /= Hkv;
  const int b = rest % n_seq, kt = rest / n_seq;        // longest tiles first
  const int grp = H / Hkv;
  const int nqt = S / AT, n_it = grp * (nqt - kt);      // query tiles from the keys' own on
  const int64_t ldq = int64_t(H) * DH, ldk = int64_t(Hkv) * DH;
  const int64_t row0 = int64_t(b) * S;
  const int key_w = kt * AT + 16 * wave;                // this wave's first key
  const float sc = 1.4426950408889634f / sqrtf(float(DH));
  const float rs = 1.0f / sqrtf(float(DH));

  const int64_t okv = (row0 + key_w + fr) * ldk + int64_t(g) * DH;
  bf16x8_t kf[KS], vf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    kf[ks] = load_frag(K + okv + 32 * ks + 8 * fk);
    vf[ks] = load_frag(V + okv + 32 * ks + 8 * fk);
  }
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    settle(kf[ks]);
    settle(vf[ks]);
  }
  f32x4_t adk[JD], adv[JD];
#pragma unroll
  for (int j = 0; j < JD; ++j) adk[j] = adv[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const uint32_t off = tile_off<DH>(wave, lane, ldq);
  float4 psr{};
  float2 dmr{};
  // the next (query head, query tile): Q, dO, LSE and D
  int fh = g * grp, ft = kt;
  auto fetch = [&](int buf) {
    const int64_t r = row0 + int64_t(ft) * AT, o = r * ldq + int64_t(fh) * DH;
    tile_dma<DH>(Q + o, ldq, off, lds_byte(sT[buf]), wave);
    tile_dma<DH>(dO + o, ldq, off, lds_byte(sT[buf] + NT), wave);
    const int64_t i = int64_t(fh) * T + r;
    if (wave == 0) dma4(LSE + i, 4u * lane, lds_byte(sL[buf]));
    if (wave == 1) dma4(Dl + i, 4u * lane, lds_byte(sD[buf]));
    if constexpr (QP) {
      if (tid < AT) {
        psr = pstat[i + tid];
        dmr = dmm[i + tid];
      }
    }
    if (++ft == nqt) {
      ft = kt;
      ++fh;
    }
  };
  fetch(0);
  int qt = kt;
  for (int it = 0; it < n_it; ++it) {
    const int buf = it & 1;
    if constexpr (QP) {
      if (tid < AT) {
        const QParams prm = make_qparams(psr.x, psr.y, 1.0f, 1.0f, qmax);
        sQh[buf][tid] = prm.h;
        sQr[buf][tid] = prm.r;
        sQz[buf][tid] = prm.z;
        sDmx[buf][tid] = dmr.x;
        sDmn[buf][tid] = dmr.y;
        sAmx[buf][tid] = __float_as_int(psr.z);
        sAmn[buf][tid] = __float_as_int(psr.w);
      }
    }
    bwd_wait();
    __syncthreads();
    if (it + 1 < n_it) fetch(buf ^ 1);                   // in flight meanwhile
    const int q0 = qt * AT;
    const bool diag = qt == kt;
    if (++qt == nqt) qt = kt;
    const uint4* tq = sT[buf];
    const uint4* to = tq + NT;
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      uint32_t wp[4], wh[4], wl[4];
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        // S and dP [16 queries x 16 keys]: lane holds queries ql + r, key fr
        const int row = 32 * k2 + row_of(hf, fr), ql = 32 * k2 + 8 * fk + 4 * hf;
        f32x4_t st = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          st = mfma(row_frag<DH>(tq, row, 4 * ks + fk), kf[ks], st);
          dp = mfma(row_frag<DH>(to, row, 4 * ks + fk), vf[ks], dp);
        }
        const f32x4_t L = lds4<f32x4_t>(&sL[buf][ql]), D = lds4<f32x4_t>(&sD[buf][ql]);
        float p[4], ds[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(fmaf(st[r], sc, -L[r]));
        f32x4_t qh, qr, qz, gmx, gmn;
        i32x4_t imx, imn;
        if constexpr (QP) {
          qh = lds4<f32x4_t>(&sQh[buf][ql]);
          qr = lds4<f32x4_t>(&sQr[buf][ql]);
          qz = lds4<f32x4_t>(&sQz[buf][ql]);
          gmx = lds4<f32x4_t>(&sDmx[buf][ql]);
          gmn = lds4<f32x4_t>(&sDmn[buf][ql]);
          imx = lds4<i32x4_t>(&sAmx[buf][ql]);
          imn = lds4<i32x4_t>(&sAmn[buf][ql]);
        }
        const int key = key_w + fr;
        if (diag) {
#pragma unroll
          for (int r = 0; r < 4; ++r) p[r] = key > q0 + ql + r ? 0.0f : p[r];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (QP) {
            QParams prm{};
            prm.h = qh[r];
            prm.r = qr[r];
            prm.z = qz[r];
            const QElem qe = quant_elem(p[r], prm, qmax);
            float gp = qe.m ? dp[r] : 0.0f;
            if (key == imx[r]) gp += gmx[r];
            if (key == imn[r]) gp += gmn[r];
            ds[r] = p[r] * (gp - D[r]) * rs;
            p[r] = dequant(qe.q, prm);                   // P^ enters dV
          } else {
            ds[r] = p[r] * (dp[r] - D[r]) * rs;  // (1/sqrt(d) of the logits)
          }
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          wp[2 * hf + e] = pack2(p[2 * e], p[2 * e + 1]);
          // dS as two bf16 terms (hi + lo, 16 significant bits): a component
          // shared by all queries' Q rows would otherwise meet its rounding
          split2(ds[2 * e], ds[2 * e + 1], &wh[2 * hf + e], &wl[2 * hf + e]);
        }
      }
      const bf16x8_t bp = bits_as_bf16x8(make_uint4(wp[0], wp[1], wp[2], wp[3]));
      const bf16x8_t bh = bits_as_bf16x8(make_uint4(wh[0], wh[1], wh[2], wh[3]));
      const bf16x8_t bl = bits_as_bf16x8(make_uint4(wl[0], wl[1], wl[2], wl[3]));
#pragma unroll
      for (int j = 0; j < JD; ++j) {
        adv[j] = mfma(col_frag<DH>(to, k2, j, lane), bp, adv[j]);
        const bf16x8_t aq = col_frag<DH>(tq, k2, j, lane);
        adk[j] = mfma(aq, bl, mfma(aq, bh, adk[j]));
      }
    }
  }
  // lane holds dK/dV[key_w + fr][16 j + 4 fk + r]
#pragma unroll
  for (int j = 0; j < JD; ++j) {
    store4(dK + okv + 4 * fk + 16 * j, adk[j]);
    store4(dV + okv + 4 * fk + 16 * j, adv[j]);
  }
}

// dQ: one workgroup per 64 queries of a head, four waves of 16.  S^T and dP^T
// as [keys x queries] tiles: a lane's values all belong to one query.  A first
// sweep over the key tiles forms D = sum_j P_ij dP_ij from the very
// probabilities the gradients use (so every row of dS sums to zero to fp32
// rounding) and writes it for the dK/dV kernel; the second sweep accumulates
// dQ^T = K^T dS^T, dS from the lane's registers as two bf16 terms.
// QP (softmax quantisation): the first sweep also forms Q_a's row sums
// S_h = sum dP^ ((q - z) - m u), S_z = sum dP^ (1 - m) and E = sum P m dP^,
// hence the row's max / min gradients (written to dmm for the dK/dV kernel)
// and D = E + max dmax + min dmin; the second sweep's dP follows Q_a's
// straight-through rule.
template <int DH, bool QP>
__global__ __launch_bounds__(ANT, 2) void attn_bwd_dq_kernel(
    const bf16raw* __restrict__ Q, const bf16raw* __restrict__ K, const bf16raw* __restrict__ V,
    const bf16raw* __restrict__ dO, const float* __restrict__ LSE, float* __restrict__ Dl,
    int S, int H, int Hkv, int n_seq, int64_t T, float* __restrict__ dQ, int p_bits,
    const float4* __restrict__ pstat, float2* __restrict__ dmm) {
  constexpr int KS = DH / 32, JD = DH / 16;
  constexpr int NT = AT * DH / 8;                        // 16-byte chunks of a tile
  __shared__ uint4 sT[2][2 * NT];                       // K, then V
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int fr = lane & 15, fk = lane >> 4;
  const AttnTile at = attn_tile(H, n_seq, S / AT);
  const int qt = at.qt, h = at.h, b = at.b;
  const int g = h / (H / Hkv);
  const int64_t ldq = int64_t(H) * DH, ldk = int64_t(Hkv) * DH;
  const int64_t row0 = int64_t(b) * S;
  const int q_w = qt * AT + 16 * wave, qrow = q_w + fr;   // this wave's first query, the lane's
  const float sc = 1.4426950408889634f / sqrtf(float(DH));
  const float rs = 1.0f / sqrtf(float(DH));
  const float qmax = QP ? float((1 << p_bits) - 1) : 0.0f;

  const int64_t oq = (row0 + qrow) * ldq + int64_t(h) * DH;
  const int64_t ri = int64_t(h) * T + row0 + qrow;
  bf16x8_t qf[KS], df[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    qf[ks] = load_frag(Q + oq + 32 * ks + 8 * fk);
    df[ks] = load_frag(dO + oq + 32 * ks + 8 * fk);
  }
  float lse = LSE[ri];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    settle(qf[ks]);
    settle(df[ks]);
  }
  settle(lse);
  // QP: Q_a's parameters of the lane's row, the row's max / min and the keys
  // that take their gradients
  QParams pr{};
  float gmx = 0.f, gmn = 0.f;
  float4 p4{};
  if constexpr (QP) {
    p4 = pstat[ri];
    pr = make_qparams(p4.x, p4.y, 1.0f, 1.0f, qmax);
  }
  f32x4_t adq[JD];
#pragma unroll
  for (int j = 0; j < JD; ++j) adq[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int nk = qt + 1;                                 // key tiles up to the diagonal
  const uint32_t off = tile_off<DH>(wave, lane, ldk);
  auto fetch = [&](int t, int buf) {
    const int64_t o = (row0 + int64_t(t) * AT) * ldk + int64_t(g) * DH;
    tile_dma<DH>(K + o, ldk, off, lds_byte(sT[buf]), wave);
    tile_dma<DH>(V + o, ldk, off, lds_byte(sT[buf] + NT), wave);
  };
  // P^T and dP^T of 16 keys of the staged tile: the tile row that accumulator
  // row fr stands for, and the key (in the sample) of this lane's first value;
  // the lane holds keys key + r, query qrow
  auto probs = [&](int buf, int row, int key, bool diag, float (&p)[4], f32x4_t& dp) {
    f32x4_t st = {0.f, 0.f, 0.f, 0.f};
    dp = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      st = mfma(row_frag<DH>(sT[buf], row, 4 * ks + fk), qf[ks], st);
      dp = mfma(row_frag<DH>(sT[buf] + NT, row, 4 * ks + fk), df[ks], dp);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(fmaf(st[r], sc, -lse));
    if (diag) {
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = key + r > qrow ? 0.0f : p[r];
    }
  };
  fetch(0, 0);
  // sweep 1: D (with QP, Q_a's row sums first); one sum per residue of the key
  // index mod 16, added up as a tree over the residue's bits
  f32x4_t dlr = {0.f, 0.f, 0.f, 0.f}, shr = dlr, szr = dlr;
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    bwd_wait();
    __syncthreads();
    fetch(kt + 1 < nk ? kt + 1 : 0, buf ^ 1);             // in flight meanwhile
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float p[4];
      f32x4_t dp;
      probs(buf, 16 * i + d_row(fr), kt * AT + 16 * i + d_row(4 * fk), kt == qt, p, dp);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if constexpr (QP) {
          const QElem qe = quant_elem(p[r], pr, qmax);
          const float t = qe.q - pr.z;
          shr[r] += dp[r] * (qe.m ? t - qe.u : t);
          szr[r] += qe.m ? 0.0f : dp[r];
          dlr[r] += qe.m ? p[r] * dp[r] : 0.0f;
        } else {
          dlr[r] += p[r] * dp[r];
        }
      }
    }
  }
  // residue bits 0 and 1 are r; bit 2 changes with fk ^ 3, bit 3 with fk ^ 1
  auto row_sum = [](f32x4_t v) {
    float x = (v[0] + v[1]) + (v[2] + v[3]);
    x += __shfl_xor(x, 48);
    return x + __shfl_xor(x, 16);
  };
  float dl = row_sum(dlr);
  if constexpr (QP) {
    const QGrad qg = quant_group_grad(row_sum(shr), row_sum(szr), p4.x, p4.y, pr, qmax);
    dl += p4.x * qg.dmx + p4.y * qg.dmn;
    gmx = qg.dmx;
    gmn = qg.dmn;
    if (fk == 0) dmm[ri] = make_float2(gmx, gmn);
  }
  if (fk == 0) Dl[ri] = dl;
  // sweep 2: dS = P (dP - D) as hi + lo bf16 terms: each row of dS sums to
  // zero, so a component shared by all K rows cancels in the exact product and
  // must not survive the rounding of dS
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = (nk + kt) & 1;
    bwd_wait();
    __syncthreads();
    if (kt + 1 < nk) fetch(kt + 1, buf ^ 1);
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      uint32_t wh[4], wl[4];
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const int key = kt * AT + 32 * k2 + 8 * fk + 4 * hf;
        float p[4], ds[4];
        f32x4_t dp;
        probs(buf, 32 * k2 + row_of(hf, fr), key, kt == qt, p, dp);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float gp = dp[r];
          if constexpr (QP) {
            gp = quant_elem(p[r], pr, qmax).m ? gp : 0.0f;
            if (key + r == __float_as_int(p4.z)) gp += gmx;
            if (key + r == __float_as_int(p4.w)) gp += gmn;
          }
          ds[r] = p[r] * (gp - dl) * rs;
        }
#pragma unroll
        for (int e = 0; e < 2; ++e)
          split2(ds[2 * e], ds[2 * e + 1], &wh[2 * hf + e], &wl[2 * hf + e]);
      }
      const bf16x8_t bh = bits_as_bf16x8(make_uint4(wh[0], wh[1], wh[2], wh[3]));
      const bf16x8_t bl = bits_as_bf16x8(make_uint4(wl[0], wl[1], wl[2], wl[3]));
      // dQ^T += K^T dS^T: A = rows of d, k = keys
#pragma unroll
      for (int j = 0; j < JD; ++j) {
        const bf16x8_t ak = col_frag<DH>(sT[buf], k2, j, lane);
        adq[j] = mfma(ak, bl, mfma(ak, bh, adq[j]));
      }
    }
  }
  // lane holds dQ[qrow][16 j + 4 fk + r]
#pragma unroll
  for (int j = 0; j < JD; ++j) store4(dQ + oq + 4 * fk + 16 * j, adq[j]);
}

template <int DH>
hipError_t attn_fwd_t(const void* Q, const void* K, const void* V, int64_t T, int S, int H,
                      int Hkv, int p_bits, float* O, float* LSE, float4* pstat, hipStream_t st) {
  const dim3 grid(unsigned(T / AT * H));
  const auto q = static_cast<const bf16raw*>(Q);
  const auto k = static_cast<const bf16raw*>(K);
  const auto v = static_cast<const bf16raw*>(V);
  if (p_bits < 16)
    hipLaunchKernelGGL(attn_fwd_q_kernel<DH>, grid, dim3(ANT), 0, st, q, k, v, S, H, Hkv, p_bits,
                       O, LSE, pstat, T);
  else if (S % (2 * AT) == 0)
    hipLaunchKernelGGL(attn_fwd2_kernel<DH>, dim3(unsigned(T / (2 * AT) * H)), dim3(ANT), 0, st, q, k, v, S, H, Hkv, O, LSE, T);
  else
    hipLaunchKernelGGL(attn_fwd_kernel<DH>, grid, dim3(ANT), 0, st, q, k, v, S, H, Hkv, O, LSE, T);
  return hipGetLastError();
}

template <int DH, bool QP>
void attn_bwd_launch(const void* Q, const void* K, const void* V, const void* dO,
                     const float* LSE, const float4* pstat, int64_t T, int S, int H, int Hkv,
                     int p_bits, float* Dl, float2* dmm, float* dQ, float* dK, float* dV,
                     hipStream_t st) {
  const auto q = static_cast<const bf16raw*>(Q);
  const auto k = static_cast<const bf16raw*>(K);
  const auto v = static_cast<const bf16raw*>(V);
  const auto o = static_cast<const bf16raw*>(dO);
  const int n_seq = int(T / S);
  // dQ first: it also writes D (and, quantised, the max / min gradients),
  // which the dK/dV kernel reads
  hipLaunchKernelGGL((attn_bwd_dq_kernel<DH, QP>), dim3(unsigned(T / AT * H)), dim3(ANT), 0, st,
                     q, k, v, o, LSE, Dl, S, H, Hkv, n_seq, T, dQ, p_bits, pstat, dmm);
  hipLaunchKernelGGL((attn_bwd_dkv_kernel<DH, QP>), dim3(unsigned(T / AT * Hkv)), dim3(ANT), 0,
                     st, q, k, v, o, LSE, Dl, S, H, Hkv, n_seq, T, dK, dV, p_bits, pstat, dmm);
}

template <int DH>
hipError_t attn_bwd_t(const void* Q, const void* K, const void* V, const void* dO,
                      const float* LSE, const float4* pstat, int64_t T, int S, int H, int Hkv,
                      int p_bits, float* ws, float* dQ, float* dK, float* dV, hipStream_t st) {
  float2* dmm = reinterpret_cast<float2*>(ws + T * H);
  if (p_bits < 16)
    attn_bwd_launch<DH, true>(Q, K, V, dO, LSE, pstat, T, S, H, Hkv, p_bits, ws, dmm, dQ, dK, dV, st);
  else
    attn_bwd_launch<DH, false>(Q, K, V, dO, LSE, nullptr, T, S, H, Hkv, 16, ws, nullptr, dQ, dK, dV,
                               st);
  return hipGetLastError();
}

}  // namespace

bool attn_supported(int64_t T, int S, int H, int Hkv, int dh) {
  return (dh == 64 || dh == 128) && S > 0 && S % AT == 0 && T > 0 && T % S == 0 && H > 0 &&
         Hkv > 0 && H % Hkv == 0 && T / S <= 65535 && H <= 65535;
}

size_t attn_bwd_ws_floats(int64_t T, int H, int p_bits) {
  return size_t(T) * size_t(H) * (p_bits < 16 ? 3 : 1);
}

hipError_t attn_fwd(const void* Q, const void* K, const void* V, int64_t T, int S, int H, int Hkv,
                    int dh, int p_bits, float* O, float* LSE, float* pstat, hipStream_t st) {
  if (!attn_supported(T, S, H, Hkv, dh)) return hipErrorInvalidValue;
  float4* ps = reinterpret_cast<float4*>(pstat);
  return dh == 128 ? attn_fwd_t<128>(Q, K, V, T, S, H, Hkv, p_bits, O, LSE, ps, st)
                   : attn_fwd_t<64>(Q, K, V, T, S, H, Hkv, p_bits, O, LSE, ps, st);
}

hipError_t attn_bwd(const void* Q, const void* K, const void* V, const void* dO, const float* LSE,
                    const float* pstat, int64_t T, int S, int H, int Hkv, int dh, int p_bits,
                    float* ws, float* dQ, float* dK, float* dV, hipStream_t st) {
  if (!attn_supported(T, S, H, Hkv, dh)) return hipErrorInvalidValue;
  const float4* ps = reinterpret_cast<const float4*>(pstat);
  return dh == 128 ? attn_bwd_t<128>(Q, K, V, dO, LSE, ps, T, S, H, Hkv, p_bits, ws, dQ, dK, dV, st)
                   : attn_bwd_t<64>(Q, K, V, dO, LSE, ps, T, S, H, Hkv, p_bits, ws, dQ, dK, dV, st);
}

}  // namespace oq
