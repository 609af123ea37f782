// fp32 storage path on gfx950's fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: exact fp32 products and sums, 256 flop per clock
// and CU, the rate of the vector ALU at its best).  Every product is held
// and accumulated in fp32, there are no atomics, and every output is bitwise
// reproducible.
//
// Paper equations: forward H = softmax(S) V with the causal mask (App. A.1);
// backward dV = P^T dO, dP = dO V^T, dS = P * (dP - rowsum(dP * P)),
// dQ = dS K / sqrt(d), dK = dS^T Q / sqrt(d) (App. A.2-A.4), evaluated per
// segment tile so prefix and suffix keys are read in place.
//
// What bounds it: the matrix instruction, 32 cycles for a 16 x 16 x 4 block.
// One 16-byte LDS read feeds four of them and one 4-byte read feeds one, so
// LDS and the vector ALU stay far below their rates and the kernels only
// need enough waves to cover latency: two workgroups of four waves per CU,
// 64 KB of double-buffered 32-row tiles each.  16-wide blocks (instead of
// 32 x 32 x 2) halve the registers a row or key costs, so a small group
// still spreads over the chip.  Measured on 32/8 heads, d = 128, P = 1000 and
// four ragged suffixes, per pass: one thread per row or key on the vector ALU
// 72.1 ms (0.9 TFLOP/s), this form 1.22 ms (54 TFLOP/s useful; the recompute of
// S and dP for dQ puts 1.3 times that through the matrix cores).
//
// v_mfma_f32_16x16x4_f32 operands (lane l, n = l % 16, g = l / 16):
//   A (16 x 4): A[n][g]   B (4 x 16): B[g][n]   C: element e = C[4 g + e][n]
// Only the pairing of A's and B's k matters.  Products over d take k = d in
// the order 16 j + 4 g + c (four consecutive floats of a row per lane, one
// 16-byte read for the steps c = 0..3); products over the rows of a C result
// take step e's k = row 4 g + e, so P and dS never leave the registers and
// the other operand is read from its row-major tile as A[n] = T[4 g + e][n].
//
// LDS tiles: 32 rows x D floats, 16-byte chunk c of row m at c ^ (m & 15):
// both reads are then free of bank conflicts (16 rows at one chunk; four
// rows 4 g + e at 64 bytes each).  Filled by direct-to-LDS loads one tile
// ahead (tile.hpp); rows past the end repeat the last one and are masked.
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "launch.hpp"
#include "tile.hpp"

namespace spr {

namespace {

constexpr int kF32Row = 16;   // rows of a wave of a query-outer workgroup
constexpr int kF32Tile = 32;  // rows of an LDS tile
constexpr int kF32BK = 32;    // keys per key-outer workgroup

__device__ __forceinline__ f32x4 mfma16(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float rounded_product(float a, float b) {
#pragma clang fp contract(off)
  return a * b;
}
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }

// One wave's share (a quarter) of a 32-row tile's direct-to-LDS loads.
template <int D>
struct F32Loader {
  static constexpr int CH = D / 4;     // 16-byte chunks per row
  static constexpr int RPI = 64 / CH;  // rows per 1 KB instruction
  static constexpr int IPW = kF32Tile / RPI / 4;
  unsigned off[IPW];
  int lrow0, lane_row;
  __device__ __forceinline__ void init(int H, int w, int lane) {
    lrow0 = w * IPW * RPI;
    lane_row = lane / CH;
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const int lrow = lrow0 + i * RPI + lane_row;
      off[i] = ((unsigned)lrow * H * D + 4 * ((lane % CH) ^ (lrow & 15))) * 4;
    }
  }
  // rows row0 .. of head hh; rows at or past nvalid (>= 1) repeat the last
  __device__ __forceinline__ void load(float* tile, const float* base, int row0, int nvalid, int H, int hh) const {
    const float* sb = base + ((size_t)row0 * H + hh) * D;
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const int lrow = lrow0 + i * RPI + lane_row;
      const unsigned back = (unsigned)(lrow - min(lrow, nvalid - 1)) * H * D * 4;
      // the chunk order follows the tile row, not the row it repeats
      dma_lds16_s(off[i] - back, sb, lds_addr(tile + (lrow0 + i * RPI) * D));
    }
  }
};

// Per-lane LDS offsets (floats) of the operand reads; blocks of 16 rows add
// a multiple of 16 D and 64 columns add 64, both immediates.
template <int D>
struct F32Offsets {
  int nat[4];    // row n, columns 16 j + 4 g .. + 3: nat[j % 4] + 64 (j / 4)
  int tr[4][4];  // row 4 g + e, column 16 db + n: tr[e][db % 4] + 64 (db / 4)
  __device__ __forceinline__ void init(int lane) {
    const int n = lane & 15, g = lane >> 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) nat[j] = n * D + 4 * ((4 * j + g) ^ n);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int q = 0; q < 4; ++q) tr[e][q] = (4 * g + e) * D + 4 * ((4 * q + (n >> 2)) ^ (4 * g + e)) + (n & 3);
  }
};
template <int D>
__device__ __forceinline__ f32x4 nat_read(const float* t, const F32Offsets<D>& fo, int row0, int j) {
  return *(const f32x4*)(t + row0 * D + 64 * (j >> 2) + fo.nat[j & 3]);
}
template <int D>
__device__ __forceinline__ float tr_read(const float* t, const F32Offsets<D>& fo, int row0, int e, int db) {
  return t[row0 * D + 64 * (db >> 2) + fo.tr[e][db & 3]];
}

// A zero P or dS of a pair that the mask hides must not meet an infinite or
// NaN value of the pair's row or key in the matrix instruction (0 * Inf is
// NaN), and A's rows serve all 16 columns of B.  So where a 16-row block has
// hidden pairs and values that are not finite, its products are added one
// visible pair at a time instead.  The backward sees such a row in the block
// of S or dP that it formed from it: all 16 of its products are not finite
// either.  The forward reads V's rows once more, in diagonal and partial
// tiles only.  Measured on the group above: 1201 us a pass without this, 1204
// with it.
__device__ __forceinline__ float times_zero(const f32x4& v, float z = 0.f) {  // z, or NaN
#pragma unroll
  for (int e = 0; e < 4; ++e) z = fmaf(v[e], 0.f, z);
  return z;
}
// !extra, which the compiler cannot merge with the branch before it: as an
// else branch the matrix products would need a second set of accumulators
__device__ __forceinline__ bool otherwise(bool extra) {
  int go = extra ? 0 : 1;
  asm volatile("" : "+v"(go));
  return __builtin_amdgcn_readfirstlane(go) != 0;
}
template <int D>
__device__ __forceinline__ bool rows_finite(const float* t, const F32Offsets<D>& fo, int row0) {
  float z = 0.f;
#pragma unroll
  for (int j = 0; j < D / 16; ++j) {
    z = times_zero(nat_read<D>(t, fo, row0, j), z);
    if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // four reads in flight: registers
  }
  return __all(z == 0.f);
}
// acc[db][e] += sum over rows lo <= k < hi (0 <= k < 16) of
// T[row0 + k][16 db + 4 g + e] p_k, where p_k of this lane's column n is
// element k % 4 of lane (n, k / 4)
template <int D>
__device__ __forceinline__ void add_visible(f32x4 (&acc)[D / 16], const float* t, int row0, const f32x4& p, int lo,
                                            int hi, int n, int g) {
  // (opaque, so that nothing computed from them is kept in registers across
  // the tile loop for this rare path)
  asm volatile("" : "+v"(n), "+v"(g));
#pragma unroll 1
  for (int k = 0; k < 16; ++k) {
    const int e = k & 3;
    const float pk = __shfl(e == 0 ? p[0] : e == 1 ? p[1] : e == 2 ? p[2] : p[3], 16 * (k >> 2) + n);
    if (k < lo || k >= hi) continue;
#pragma unroll
    for (int db = 0; db < D / 16; ++db) {
      const f32x4 v = *(const f32x4*)(t + (row0 + k) * D + 4 * ((4 * db + g) ^ k));
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[db][c] = fmaf(pk, v[c], acc[db][c]);
      __builtin_amdgcn_sched_barrier(0);  // one read at a time: registers
    }
  }
}

// Query-outer workgroups in one of two forms.  KS = 1: 64 rows of one q
// head, 16 per wave, every wave takes all 32 keys of a tile.  KS = 2 (launches
// of fewer than 1024 workgroups of 64 rows, four per CU): 32 rows, waves 2 and
// 3 repeat the rows of waves 0 and 1 and each takes 16 keys of a tile, so a
// sweep's chain of products is half as long and there are twice the
// workgroups; the two key halves are merged through LDS at the end.  Measured
// on the group above: the 64-row suffix's forward 94 -> 63 us and backward
// 135 -> 87 us; the prefix forward (512 workgroups of 64 rows) 115 -> 110 us.
// Block b -> (kv head b % Hkv, q head of its group, row tile, suffix), the
// rows with the most keys first; every block of one kv head lands on one XCD
// for Hkv dividing 8.  The launch arguments count 16-row tiles.
template <int KS>
struct QForm {
  static constexpr int BQ = 4 * kF32Row / KS;  // rows per workgroup
  static constexpr int NKB = 2 / KS;           // 16-key blocks per wave and tile
  __host__ __device__ static int tiles(int tiles16) { return (tiles16 + 4 / KS - 1) / (4 / KS); }
};
struct F32Rows {
  bool prefix;
  int lp0, seg_len, row_base, hq, hk;
};
template <int KS>
__device__ __forceinline__ bool decode_rows(const AttnArgs& a, int bid, int n_blocks, F32Rows& t) {
  const int G = a.hq / a.hkv, ntp = QForm<KS>::tiles(a.n_prefix_q_tiles);
  const int ntx = ntp + QForm<KS>::tiles(a.n_suffix_q_tiles);
  int b = bid;
  t.hk = b % a.hkv;
  b /= a.hkv;
  t.hq = t.hk * G + b % G;
  b /= G;
  const int tile = causal_tile_order(b % ntx, ntx, a.hq, n_blocks);
  if (tile < ntp) {
    t.prefix = true;
    t.lp0 = tile * QForm<KS>::BQ;
    t.seg_len = a.P;
    t.row_base = 0;
  } else {
    t.prefix = false;
    t.lp0 = (tile - ntp) * QForm<KS>::BQ;
    const SegRows sg = suffix_rows(a.cu, a.seq_base + b / ntx, a.total_len);
    t.row_base = sg.base;
    t.seg_len = sg.len;
  }
  return t.lp0 < t.seg_len;
}

// The key tiles a query-outer workgroup sweeps: prefix keys (causal for
// prefix rows), then the suffix's own.
struct F32Keys {
  int nkeys0, nkeys1, nt0, nt;
  __device__ __forceinline__ F32Keys(const AttnArgs& a, const F32Rows& t, int bq) {
    const int last = min(t.lp0 + bq, t.seg_len) - 1;
    nkeys0 = t.prefix ? min(a.P, last + 1) : a.P;
    nkeys1 = t.prefix ? 0 : last + 1;
    nt0 = (nkeys0 + kF32Tile - 1) / kF32Tile;
    nt = nt0 + (nkeys1 + kF32Tile - 1) / kF32Tile;
  }
};

// Sweeps the key tiles of a query-outer workgroup, double-buffered:
// step(k0, nk, causal, K tile, V tile) for each.
template <int D, int KS, typename Step>
__device__ __forceinline__ void sweep_keys(const AttnArgs& a, const F32Rows& t, int w, int lane,
                                           float (*Ks)[kF32Tile * D], float (*Vs)[kF32Tile * D], Step step) {
  const F32Keys ks(a, t, QForm<KS>::BQ);
  const float *k_p = in_sgpr((const float*)a.k_p), *k_s = in_sgpr((const float*)a.k_s);
  const float *v_p = in_sgpr((const float*)a.v_p), *v_s = in_sgpr((const float*)a.v_s);
  F32Loader<D> ld;
  ld.init(a.hkv, w, lane);
  auto issue = [&](int i) {
    const bool p = i < ks.nt0;
    const int k0 = (p ? i : i - ks.nt0) * kF32Tile;
    const int nk = min(kF32Tile, (p ? ks.nkeys0 : ks.nkeys1) - k0), row = (p ? 0 : t.row_base) + k0;
    ld.load(Ks[i & 1], pick(p, k_p, k_s), row, nk, a.hkv, t.hk);
    ld.load(Vs[i & 1], pick(p, v_p, v_s), row, nk, a.hkv, t.hk);
  };
  if (ks.nt > 0) issue(0);
  tile_barrier();
  for (int i = 0; i < ks.nt; ++i) {
    if (i + 1 < ks.nt) issue(i + 1);
    compiler_fence();
    const bool p = i < ks.nt0;
    const int k0 = (p ? i : i - ks.nt0) * kF32Tile;
    step(k0, min(kF32Tile, (p ? ks.nkeys0 : ks.nkeys1) - k0), p == t.prefix, Ks[i & 1], Vs[i & 1]);
    tile_barrier();
  }
}

}  // namespace

// ---------------------------------------------------------------- forward
// S^T = K Q^T with lane (n, g) holding four keys of row n per block, so a
// row's softmax statistics take two shuffles; O^T += V^T P^T.
template <int D, int KS>
__global__ __launch_bounds__(kThreads, 2) void fwd_f32_kernel(AttnArgs a) {
  constexpr int NJ = D / 16, NKB = QForm<KS>::NKB;
  __shared__ __attribute__((aligned(1024))) float Ks[2][kF32Tile * D];
  __shared__ __attribute__((aligned(1024))) float Vs[2][kF32Tile * D];
  F32Rows t;
  if (!decode_rows<KS>(a, blockIdx.x, gridDim.x, t)) return;
  const int lane = threadIdx.x & 63, w = wave_id(), n = lane & 15, g = lane >> 4;
  F32Offsets<D> fo;
  fo.init(lane);
  const int ks = KS == 2 ? w >> 1 : 0;  // key half of the tile
  const int wave_lp0 = t.lp0 + kF32Row * (KS == 2 ? w & 1 : w), lp = wave_lp0 + n;
  const int my_lp = min(lp, t.seg_len - 1);  // rows past the end recompute the last one
  f32x4 q[NJ], o[NJ];
  const size_t off = ((size_t)(t.row_base + my_lp) * a.hq + t.hq) * D + 4 * g;
  {
    const float* qb = (const float*)(t.prefix ? a.q_p : a.q_s);
#pragma unroll
    for (int j = 0; j < NJ; ++j) q[j] = *(const f32x4*)(qb + off + 16 * j);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      settle(q[j]);
      o[j] = zero4();
    }
  }
  float m = -INFINITY, l = 0.f;  // running max (log2 domain); this lane's share of the row sum

  sweep_keys<D, KS>(a, t, w, lane, Ks, Vs, [&](int k0, int nk, bool causal, const float* Kc, const float* Vc) {
    const int kk = k0 + 16 * ks;  // this wave's first key
    if (wave_lp0 >= t.seg_len || (causal && kk > wave_lp0 + 15)) return;  // no row of this wave sees them
    f32x4 st[2] = {zero4(), zero4()};  // st[b][e] = S^T[key kk + 16 b + 4 g + e][row n]
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      // two independent chains: the tile's two key blocks, or the even and
      // odd j of the one block
      const f32x4 k_0 = nat_read<D>(Kc, fo, 16 * ks, j), k_1 = NKB == 2 ? nat_read<D>(Kc, fo, 16, j) : k_0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (NKB == 2 || j % 2 == 0) st[0] = mfma16(k_0[c], q[j][c], st[0]);
        if (NKB == 2 || j % 2 == 1) st[1] = mfma16(k_1[c], q[j][c], st[1]);
      }
    }
    if (NKB == 1) st[0] += st[1];
    const bool masked = nk < kF32Tile || (causal && k0 + kF32Tile - 1 > wave_lp0);
    const int hi = (causal ? min(nk, my_lp - k0 + 1) : nk) - 16 * ks;  // keys kk .. kk + hi - 1 are visible
    if (masked) {
      const int lim = hi - 4 * g;
#pragma unroll
      for (int i = 0; i < 4 * NKB; ++i)
        st[i >> 2][i & 3] = 16 * (i >> 2) + (i & 3) < lim ? st[i >> 2][i & 3] : -INFINITY;
    }
    float mt = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4 * NKB; ++i) mt = fmaxf(mt, st[i >> 2][i & 3]);
    mt = fmaxf(mt, __shfl_xor(mt, 16));
    mt = fmaxf(mt, __shfl_xor(mt, 32)) * a.scale_log2;
    if (__any(mt > m)) {
      const float mn = fmaxf(m, mt);
      const float corr = exp2f(m - (mn == -INFINITY ? 0.f : mn));
      l *= corr;
#pragma unroll
      for (int j = 0; j < NJ; ++j) o[j] *= corr;
      m = mn;
    }
    const float mu = m == -INFINITY ? 0.f : m;
    // The fused product differs from the rounded one in m by up to 2^-25 |m|.
    // That cancels between O, l and the LSE as long as 2^(2^-25 |m|) is in
    // range; beyond, the products are rounded alike.
    if (__builtin_expect(__any(fabsf(mu) > 0x1p30f), 0)) {
#pragma unroll
      for (int i = 0; i < 4 * NKB; ++i) st[i >> 2][i & 3] = exp2f(rounded_product(st[i >> 2][i & 3], a.scale_log2) - mu);
    } else {
#pragma unroll
      for (int i = 0; i < 4 * NKB; ++i) st[i >> 2][i & 3] = exp2f(fmaf(st[i >> 2][i & 3], a.scale_log2, -mu));
    }
#pragma unroll
    for (int i = 0; i < 4 * NKB; ++i) l += st[i >> 2][i & 3];
#pragma unroll
    for (int b = 0; b < NKB; ++b) {
      const bool extra = masked && !rows_finite<D>(Vc, fo, 16 * (ks + b));
      if (__builtin_expect(extra, 0)) add_visible<D>(o, Vc, 16 * (ks + b), st[b], 0, hi - 16 * b, n, g);
      if (!otherwise(extra)) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int db = 0; db < NJ; ++db)
          o[db] = mfma16(tr_read<D>(Vc, fo, 16 * (ks + b), e, db), st[b][e], o[db]);
    }
  });

  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if constexpr (KS == 2) {
    // merge the key halves: waves 2 and 3 hand over max, sum and O
    f32x4* xo = (f32x4*)Ks;  // [wave][db][lane]; the tiles are no longer read
    float* xm = (float*)Vs;  // [wave][max, sum][lane]
    const int r = w & 1;
    if (ks == 1) {
      xm[128 * r + lane] = m;
      xm[128 * r + 64 + lane] = l;
#pragma unroll
      for (int db = 0; db < NJ; ++db) xo[(r * NJ + db) * 64 + lane] = o[db];
    }
    __syncthreads();
    if (ks == 1) return;
    const float m1 = xm[128 * r + lane], l1 = xm[128 * r + 64 + lane];
    const float mn = fmaxf(m, m1), mu = mn == -INFINITY ? 0.f : mn;  // (every visible score -Inf)
    const float c0 = exp2f(m - mu), c1 = exp2f(m1 - mu);
    l = l * c0 + l1 * c1;
#pragma unroll
    for (int db = 0; db < NJ; ++db) o[db] = o[db] * c0 + xo[(r * NJ + db) * 64 + lane] * c1;
    m = mn;
  }
  if (lp >= t.seg_len) return;
  const float inv = 1.f / l;
  float* ob = (float*)(t.prefix ? a.o_p : a.o_s);
#pragma unroll
  for (int db = 0; db < NJ; ++db) *(f32x4*)(ob + off + 16 * db) = o[db] * inv;
  if (g == 0) (t.prefix ? a.lse_p : a.lse_s)[(size_t)(t.row_base + lp) * a.hq + t.hq] = (m + log2f(l)) * kLn2;
}

namespace {

// ------------------------------------------------------- backward, dK / dV
template <int D>
struct F32KvLds {
  float q[2][kF32Tile * D], o[2][kF32Tile * D];
  float l[2][64], e[2][64];  // log2-domain LSE and rowsum(dO * O) of the tile's rows (32 used)
};

// Key-outer: 32 keys of one kv head per workgroup, sweeping every row that
// sees them, for all G q heads, in 32-row tiles.  Wave w takes keys
// 16 (w % 2) and rows 16 (w / 2) of each tile; the two row halves' sums are
// added through LDS at the end (one wave finishes dV, the other dK).
template <int D>
__device__ __forceinline__ void bwd_kv_f32(const AttnArgs& a, int bid, F32KvLds<D>& L) {
  constexpr int NJ = D / 16;
  const int lane = threadIdx.x & 63, w = wave_id(), n = lane & 15, g = lane >> 4;
  const int kb = w & 1, rh = w >> 1;
  F32Offsets<D> fo;
  fo.init(lane);
  const int R = a.kv_rsplit > 1 ? a.kv_rsplit : 1;
  const int G = a.hq / a.hkv, hk = bid % a.hkv, rs = (bid / a.hkv) % R, x = bid / a.hkv / R;
  bool kpre;
  int k0, kseg, kbase;
  if (x < a.n_prefix_k_tiles) {
    kpre = true;
    k0 = x * kF32BK;
    kseg = a.P;
    kbase = 0;
  } else {
    const int y = x - a.n_prefix_k_tiles;
    kpre = false;
    k0 = (y % a.n_suffix_k_tiles) * kF32BK;
    const SegRows sg = suffix_rows(a.cu, a.seq_base + y / a.n_suffix_k_tiles, a.total_len);
    kbase = sg.base;
    kseg = sg.len;
  }
  if (k0 >= kseg) return;
  const int wave_k0 = k0 + 16 * kb, key = wave_k0 + n;
  const int my_key = min(key, kseg - 1);  // keys past the end recompute the last one
  f32x4 kf[NJ], vf[NJ], dk[NJ], dv[NJ];
  {
    const float* kg = (const float*)(kpre ? a.k_p : a.k_s);
    const float* vg = (const float*)(kpre ? a.v_p : a.v_s);
    const size_t off = ((size_t)(kbase + my_key) * a.hkv + hk) * D + 4 * g;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      kf[j] = *(const f32x4*)(kg + off + 16 * j);
      vf[j] = *(const f32x4*)(vg + off + 16 * j);
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      settle(kf[j]);
      settle(vf[j]);
      dk[j] = zero4();
      dv[j] = zero4();
    }
  }
  // row tiles: a prefix key tile sees prefix rows from k0 on (causal) and/or
  // every suffix row of the launch; a suffix key tile its own rows from k0 on
  int n_pr = 0, n_sr = 0, sr0 = 0, sr1 = 0;
  if (kpre) {
    if (a.prefix_rows) n_pr = (a.P - k0 + kF32Tile - 1) / kF32Tile;
    if (a.suffix_rows) {
      const SegRows sp = suffix_span(a.cu, a.seq_base, a.seq_base + a.n_seq, a.total_len);
      sr0 = sp.base;
      sr1 = sp.base + sp.len;
      n_sr = (sp.len + kF32Tile - 1) / kF32Tile;
    }
  } else {
    n_sr = (kseg - k0 + kF32Tile - 1) / kF32Tile;
  }
  // this block's contiguous share of the (row tile, head) sequence below
  const int all = G * (n_pr + n_sr);
  const int t_lo = (int)((long)all * rs / R), nt = (int)((long)all * (rs + 1) / R) - t_lo;
  struct RowTile {
    int row0, nr, lp;  // memory row, valid rows, segment-local first row
    bool prefix, causal;
  };
  // row tiles outer, heads inner (neighbouring key tiles then read the same
  // rows at about the same time); causal ranges from the last row down
  auto info = [&](int j) {
    RowTile rt;
    if (kpre && j < n_sr) {
      rt = {sr0 + j * kF32Tile, 0, 0, false, false};
      rt.nr = min(kF32Tile, sr1 - rt.row0);
    } else if (kpre) {
      const int lp = k0 + (n_pr - 1 - (j - n_sr)) * kF32Tile;
      rt = {lp, min(kF32Tile, a.P - lp), lp, true, true};
    } else {
      const int lp = k0 + (n_sr - 1 - j) * kF32Tile;
      rt = {kbase + lp, min(kF32Tile, kseg - lp), lp, false, true};
    }
    return rt;
  };
  const float *q_p = in_sgpr((const float*)a.q_p), *q_s = in_sgpr((const float*)a.q_s);
  const float *do_p = in_sgpr((const float*)a.do_p), *do_s = in_sgpr((const float*)a.do_s);
  const float *l_p = in_sgpr((const float*)a.lse2_p), *l_s = in_sgpr((const float*)a.lse2_s);
  const float *e_p = in_sgpr((const float*)a.dd_p), *e_s = in_sgpr((const float*)a.dd_s);
  F32Loader<D> ld;
  ld.init(a.hq, w, lane);
  RowVecLoader rl;
  rl.init(a.hq, lane);
  auto issue = [&](int j, int gi, int b) {
    const RowTile rt = info(j);
    const int hh = hk * G + gi;
    ld.load(L.q[b], pick(rt.prefix, q_p, q_s), rt.row0, rt.nr, a.hq, hh);
    ld.load(L.o[b], pick(rt.prefix, do_p, do_s), rt.row0, rt.nr, a.hq, hh);
    if (w == 0) rl.load(L.l[b], pick(rt.prefix, l_p, l_s) + hh, rt.row0, rt.nr, a.hq);
    if (w == 1) rl.load(L.e[b], pick(rt.prefix, e_p, e_s) + hh, rt.row0, rt.nr, a.hq);
  };

  int lj = t_lo / G, lg = t_lo % G, cj = lj, cg = lg;  // next tile to load, next to compute
  auto next = [&](int& j, int& gi) {
    if (++gi == G) {
      gi = 0;
      ++j;
    }
  };
  if (nt > 0) {
    issue(lj, lg, 0);
    next(lj, lg);
  }
  tile_barrier();
  for (int i = 0; i < nt; ++i) {
    const int b = i & 1;
    if (i + 1 < nt) {
      issue(lj, lg, b ^ 1);
      next(lj, lg);
    }
    compiler_fence();
    const RowTile rt = info(cj);
    next(cj, cg);
    // this wave's 16 rows of the tile: any valid, any seeing its keys?
    if (16 * rh < rt.nr && !(rt.causal && rt.lp + 16 * rh + 15 < wave_k0)) {
      const float *Qc = L.q[b], *Oc = L.o[b];
      f32x4 s = zero4(), dp = zero4();  // [row 16 rh + 4 g + e][key n]
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const f32x4 qa = nat_read<D>(Qc + 16 * D * rh, fo, 0, j), oa = nat_read<D>(Oc + 16 * D * rh, fo, 0, j);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          s = mfma16(qa[c], kf[j][c], s);
          dp = mfma16(oa[c], vf[j][c], dp);
        }
      }
      const f32x4 l4 = *(const f32x4*)(L.l[b] + 16 * rh + 4 * g), e4 = *(const f32x4*)(L.e[b] + 16 * rh + 4 * g);
      // row lp + 16 rh + q sees this lane's key iff q >= q_lo (causal) and
      // q < q_hi; some pair of the block is hidden iff `masked`
      const int q_lo = (rt.causal ? my_key - rt.lp : 0) - 16 * rh, q_hi = rt.nr - 16 * rh;
      const bool masked = q_hi < 16 || (rt.causal && rt.lp + 16 * rh < wave_k0 + 15);
      const bool extra = masked && !__all(times_zero(s, times_zero(dp)) == 0.f);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool vis = 4 * g + e >= q_lo && 4 * g + e < q_hi;
        const float p = exp2f(fmaf(s[e], a.scale_log2, -l4[e]));
        s[e] = vis ? p : 0.f;
        dp[e] = vis ? p * (dp[e] - e4[e]) : 0.f;
      }
      if (__builtin_expect(extra, 0)) {
        add_visible<D>(dv, Oc, 16 * rh, s, q_lo, q_hi, n, g);
        add_visible<D>(dk, Qc, 16 * rh, dp, q_lo, q_hi, n, g);
      }
      if (otherwise(extra)) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int db = 0; db < NJ; ++db) {
            dv[db] = mfma16(tr_read<D>(Oc + 16 * D * rh, fo, 0, e, db), s[e], dv[db]);
            dk[db] = mfma16(tr_read<D>(Qc + 16 * D * rh, fo, 0, e, db), dp[e], dk[db]);
          }
      }
    }
    tile_barrier();
  }

  // the other row half's sums (the tiles are no longer read)
  f32x4* xch = (f32x4*)&L;  // [kb][rh][db][lane]
#pragma unroll
  for (int db = 0; db < NJ; ++db) xch[((kb * 2 + rh) * NJ + db) * 64 + lane] = rh == 0 ? dk[db] : dv[db];
  __syncthreads();
  if (key >= kseg) return;
  const float sc = rh == 0 ? 1.f : a.scale;  // rh 0 finishes dV, rh 1 dK
  const size_t off = ((size_t)(kbase + key) * a.hkv + hk) * D + 4 * g;
  float* cache = rh == 0 ? a.gv : a.gk;
  float* out = (float*)(rh == 0 ? (kpre ? a.dv_p : a.dv_s) : (kpre ? a.dk_p : a.dk_s));
#pragma unroll
  for (int db = 0; db < NJ; ++db) {
    const f32x4 other = xch[((kb * 2 + (rh ^ 1)) * NJ + db) * 64 + lane];
    const f32x4 v = (rh == 0 ? dv[db] + other : other + dk[db]) * sc;
    const size_t at = off + 16 * db;
    if (rs > 0)  // a later share's partial, added by kv_combine_f32_kernel
      *(f32x4*)((rh == 0 ? a.part_dv : a.part_dk) + (size_t)(rs - 1) * a.P * a.hkv * D + at) = v;
    else if (!kpre || R > 1)
      *(f32x4*)(out + at) = v;
    else if (a.pk_mode == kPkAccumulate)
      *(f32x4*)(cache + at) = *(const f32x4*)(cache + at) + v;
    else
      *(f32x4*)(out + at) = v + *(const f32x4*)(cache + at);
  }
}

// ------------------------------------------------------------ backward, dQ
// Query-outer (QForm): S^T and dP^T recomputed, dQ^T += K^T dS^T, written
// once, scaled (the dense baseline's prefix rows:
// added unscaled to its fp32 sum over the trajectories).
template <int D, int KS>
__device__ __forceinline__ void bwd_q_f32(const AttnArgs& a, int bid, float (*Ks)[kF32Tile * D],
                                          float (*Vs)[kF32Tile * D]) {
  constexpr int NJ = D / 16, NKB = QForm<KS>::NKB;
  F32Rows t;
  if (!decode_rows<KS>(a, bid, 1 << 30, t)) return;  // (beside the key-outer blocks: longest first)
  const int lane = threadIdx.x & 63, w = wave_id(), n = lane & 15, g = lane >> 4;
  F32Offsets<D> fo;
  fo.init(lane);
  const int ks = KS == 2 ? w >> 1 : 0;
  const int wave_lp0 = t.lp0 + kF32Row * (KS == 2 ? w & 1 : w), lp = wave_lp0 + n;
  const int my_lp = min(lp, t.seg_len - 1);
  const size_t rh = (size_t)(t.row_base + my_lp) * a.hq + t.hq, off = rh * D + 4 * g;
  f32x4 q[NJ], d_o[NJ], dq[NJ];
  float lse2 = (t.prefix ? a.lse2_p : a.lse2_s)[rh], drow = (t.prefix ? a.dd_p : a.dd_s)[rh];
  {
    const float* qb = (const float*)(t.prefix ? a.q_p : a.q_s);
    const float* ob = (const float*)(t.prefix ? a.do_p : a.do_s);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      q[j] = *(const f32x4*)(qb + off + 16 * j);
      d_o[j] = *(const f32x4*)(ob + off + 16 * j);
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      settle(q[j]);
      settle(d_o[j]);
      dq[j] = zero4();
    }
    settle(lse2);
    settle(drow);
  }
  sweep_keys<D, KS>(a, t, w, lane, Ks, Vs, [&](int k0, int nk, bool causal, const float* Kc, const float* Vc) {
    if (wave_lp0 >= t.seg_len || (causal && k0 + 16 * ks > wave_lp0 + 15)) return;
    f32x4 st[2] = {zero4(), zero4()}, pt[2] = {zero4(), zero4()};  // [key 16 (ks + kb) + 4 g + e][row n]
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        const f32x4 ka = nat_read<D>(Kc, fo, 16 * (ks + kb), j), va = nat_read<D>(Vc, fo, 16 * (ks + kb), j);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          st[kb] = mfma16(ka[c], q[j][c], st[kb]);
          pt[kb] = mfma16(va[c], d_o[j][c], pt[kb]);
        }
      }
    const bool masked = nk < kF32Tile || (causal && k0 + kF32Tile - 1 > wave_lp0);
    const int hi = (causal ? min(nk, my_lp - k0 + 1) : nk) - 16 * ks;  // this wave's keys 0 .. hi - 1 are visible
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
      f32x4 ds;
      const bool extra = masked && !__all(times_zero(st[kb]) == 0.f);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float p = exp2f(fmaf(st[kb][e], a.scale_log2, -lse2));
        ds[e] = 16 * kb + 4 * g + e < hi ? p * (pt[kb][e] - drow) : 0.f;
      }
      if (__builtin_expect(extra, 0)) add_visible<D>(dq, Kc, 16 * (ks + kb), ds, 0, hi - 16 * kb, n, g);
      if (!otherwise(extra)) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int db = 0; db < NJ; ++db)
          dq[db] = mfma16(tr_read<D>(Kc, fo, 16 * (ks + kb), e, db), ds[e], dq[db]);
    }
  });
  if constexpr (KS == 2) {
    // the key halves' sums, through the tiles no longer read
    f32x4* x = (f32x4*)Ks;  // [wave][db][lane]
#pragma unroll
    for (int db = 0; db < NJ; ++db)
      if (ks == 1) x[((w & 1) * NJ + db) * 64 + lane] = dq[db];
    __syncthreads();
    if (ks == 1) return;
#pragma unroll
    for (int db = 0; db < NJ; ++db) dq[db] += x[((w & 1) * NJ + db) * 64 + lane];
  }
  if (lp >= t.seg_len) return;
  if (t.prefix && a.dq_p_accumulate) {
#pragma unroll
    for (int db = 0; db < NJ; ++db) {
      f32x4* p = (f32x4*)(a.dq_acc_p + off + 16 * db);
      *p = *p + dq[db];
    }
    return;
  }
  float* out = (float*)(t.prefix ? a.dq_p : a.dq_s);
#pragma unroll
  for (int db = 0; db < NJ; ++db) *(f32x4*)(out + off + 16 * db) = dq[db] * a.scale;
}

}  // namespace

// Both roles in one launch, so that a small group's key tiles and row tiles
// share the chip: n_kv key-outer blocks first (their sweeps are the longest),
// then the query-outer ones.
template <int D, int KS>
__global__ __launch_bounds__(kThreads, 2) void bwd_f32_kernel(AttnArgs a, int n_kv) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[sizeof(F32KvLds<D>)];
  const int b = blockIdx.x;
  if (b < n_kv) {
    bwd_kv_f32<D>(a, b, *(F32KvLds<D>*)lds);
  } else {
    float(*tiles)[kF32Tile * D] = (float(*)[kF32Tile * D])lds;
    bwd_q_f32<D, KS>(a, b - n_kv, tiles, tiles + 2);
  }
}

// dK_P/dV_P of a Phase C whose key sweeps were cut into kv_rsplit shares:
// share 0 lies in the outputs themselves, the others in part_dk/part_dv; all
// are added in share order, then the cache.
__global__ __launch_bounds__(kThreads) void kv_combine_f32_kernel(AttnArgs a, size_t n4) {
  const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n4) return;
  f32x4 k = ((f32x4*)a.dk_p)[i], v = ((f32x4*)a.dv_p)[i];
  for (int j = 1; j < a.kv_rsplit; ++j) {
    k += ((const f32x4*)a.part_dk)[(j - 1) * n4 + i];
    v += ((const f32x4*)a.part_dv)[(j - 1) * n4 + i];
  }
  ((f32x4*)a.dk_p)[i] = k + ((const f32x4*)a.gk)[i];
  ((f32x4*)a.dv_p)[i] = v + ((const f32x4*)a.gv)[i];
}

// ------------------------------------------------------------- launchers
int f32_block_q() { return kF32Row; }
int f32_block_k() { return kF32BK; }

namespace {
// query-outer workgroups of a launch in form KS
template <int KS>
long q_blocks(const AttnArgs& a, int n_z) {
  return (long)(QForm<KS>::tiles(a.n_prefix_q_tiles) + QForm<KS>::tiles(a.n_suffix_q_tiles)) * a.hq * n_z;
}
// KS = 2 below four workgroups of 64 rows per CU; at two (512) it still gains
// 4% (see QForm).
constexpr long kF32SplitBelow = 1024;
}  // namespace

hipError_t launch_fwd_f32(const AttnArgs& a, int head_dim, int n_z, hipStream_t st) {
  const bool split = q_blocks<1>(a, n_z) < kF32SplitBelow;
  const dim3 grid((unsigned)(split ? q_blocks<2>(a, n_z) : q_blocks<1>(a, n_z)));
  if (grid.x == 0) return hipSuccess;
  ProfileScope ps("fwd_f32", st);
  if (head_dim == 64 && split)
    hipLaunchKernelGGL((fwd_f32_kernel<64, 2>), grid, dim3(kThreads), 0, st, a);
  else if (head_dim == 64)
    hipLaunchKernelGGL((fwd_f32_kernel<64, 1>), grid, dim3(kThreads), 0, st, a);
  else if (split)
    hipLaunchKernelGGL((fwd_f32_kernel<128, 2>), grid, dim3(kThreads), 0, st, a);
  else
    hipLaunchKernelGGL((fwd_f32_kernel<128, 1>), grid, dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_bwd_f32(const AttnArgs& a, int head_dim, int n_qz, hipStream_t st) {
  const int R = a.kv_rsplit > 1 ? a.kv_rsplit : 1;
  // shares: Phase C only (prefix keys, injected cache)
  if (R > 1 && (a.n_suffix_k_tiles || a.suffix_rows || a.pk_mode != kPkInject || !a.part_dk || !a.part_dv))
    return hipErrorInvalidValue;
  const long n_kv = ((long)a.n_prefix_k_tiles + (long)a.n_seq * a.n_suffix_k_tiles) * a.hkv * R;
  const bool split = q_blocks<1>(a, n_qz) < kF32SplitBelow;
  const long n_q = split ? q_blocks<2>(a, n_qz) : q_blocks<1>(a, n_qz);
  if (n_kv + n_q == 0) return hipSuccess;
  const dim3 grid((unsigned)(n_kv + n_q));
  ProfileScope ps("bwd_f32", st);
  if (head_dim == 64 && split)
    hipLaunchKernelGGL((bwd_f32_kernel<64, 2>), grid, dim3(kThreads), 0, st, a, (int)n_kv);
  else if (head_dim == 64)
    hipLaunchKernelGGL((bwd_f32_kernel<64, 1>), grid, dim3(kThreads), 0, st, a, (int)n_kv);
  else if (split)
    hipLaunchKernelGGL((bwd_f32_kernel<128, 2>), grid, dim3(kThreads), 0, st, a, (int)n_kv);
  else
    hipLaunchKernelGGL((bwd_f32_kernel<128, 1>), grid, dim3(kThreads), 0, st, a, (int)n_kv);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || R == 1 || n_kv == 0) return e;
  const size_t n4 = (size_t)a.P * a.hkv * head_dim / 4;
  ProfileScope pk("bwd_kv_combine", st);
  hipLaunchKernelGGL(kv_combine_f32_kernel, dim3((unsigned)((n4 + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                     a, n4);
  return hipGetLastError();
}

int f32_kvsplit(long kv_tiles, long max_tiles, int group) {
  // As bwd_bf16_kvsplit: key tile 0 sweeps every row (max_tiles 32-row steps
  // of one kv head), and it would end the launch alone where that is over
  // 10% more than a slot's average of the launch (two slots per CU, the
  // query-outer role adding three quarters of kv_tiles).  Measured at
  // P = 1000, Hq 32, Hkv 8: Phase C 417 us whole, 299 in three shares.  Share 0 goes to
  // the outputs and the workspace holds group / 2 more (prefix_bwd_parts).
  const double per_slot = 1.75 * (double)kv_tiles / 512;
  if ((double)max_tiles <= 1.1 * per_slot) return 1;
  const long r = std::min((long)std::ceil((double)max_tiles / per_slot), max_tiles / 8);
  return (int)std::max(1L, std::min(r, 1L + group / 2));
}

}  // namespace spr
