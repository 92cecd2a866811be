// fp32 GEMM on the bf16 matrix cores: every fp32 operand is taken as the sum of
// three bf16 values (8 + 8 + 8 significant bits, rounded to nearest, so the
// rest is below 2^-27 of the operand) and every product as the six partial
// products whose size is at least 2^-18 of the whole,
//   a b ~ a0 b0 + (a0 b1 + a1 b0) + (a0 b2 + a1 b1 + a2 b0),
// summed in fp32.  The dropped terms are below 2^-25 |a b|, less than the
// rounding of one fp32 product, so the results are as exact as fp32 MFMAs
// give, for operands above about 2^-109 (the third term of smaller ones falls
// below the smallest bf16 numbers, so they keep fewer bits).  The split and the
// choice of products are those of Henry, Tang and Heinecke (Leveraging the bfloat16
// Artificial Intelligence Datatype for Higher-Precision Computations, ARITH 2019).
// v_mfma_f32_32x32x16_bf16 does 16 times the flops of
// v_mfma_f32_16x16x4_f32 per cycle, so six products still leave 2.7 times.
//
// Measured (us, this kernel / gemm_f32_kernel; relative error against 64 bits):
//   4096 x 4096 x 4096                  822 / 1327   3.7e-7 / 1.2e-6
//   1024 x 256, k 10000 in 32 splits     38 / 56     1.4e-7 / 3.3e-7
//   10000 x 256, k 1024 in 3 splits      39 / 62     1.0e-7 / 4.1e-7
//   10 x 256, k 1000000 in 512 splits   177 / 590    4.2e-7 / 1.5e-6
//   10 x 1000000, k 256                 250 / 358    1.0e-7 / 2.9e-7
//   1024 x 10000, k 256, MSE epilogue    55 / 66     8.6e-8 / 2.9e-7
// 822 us are 1.0 PFLOP/s of bf16 products; torch's bf16 GEMM reaches 1.15 on the
// same card, at the 1.75 GHz that it holds under such a load.  The forward
// with k = 256 is bound by its epilogue: the blocks start together, so the
// targets' reads and the results' writes (82 MB) hardly overlap other blocks'
// products (while this kernel still spilled registers, at 63 us: targets read
// ahead of the main loop 66 us; wave priorities by block no change).
//
// Operand storage, GemmArgs, epilogues and tile order are those of
// gemm_f32_kernel.  Block: 256 threads, WGM x WGN wavefronts of (32 FM) x
// (32 FN) (accumulator element r of lane l is D[8 (r/4) + 4 (l/32) + r%4][l%32]),
// k tile 16 = one MFMA step, LDS double-buffered: while the MFMAs of tile t run,
// the fp32 values of tile t + 1 (loaded one tile earlier) are split on the
// vector units and stored, and the loads of tile t + 2 are issued.  The barrier
// waits for LDS only, so those loads stay in flight across it.
//
// LDS holds three bf16 planes per operand in the operand's own layout:
//   KMajor:  [mn][16]; a row is two 16-byte chunks, swapped for every second
//            group of 8 rows, so that 16 lanes reading 16 rows at one chunk touch 16
//            different 16-byte bank groups.
//   MNMajor: [16][mn]; read with ds_read_b64_tr_b16, chunks permuted by XOR with
//            a function of the row (4 rows x 4 chunks per half wavefront).
// With a KMajor B and FN = 2, fragment h of MFMA column j covers tile column
// 2 j + h (its rows are stored permuted), so that a lane's outputs of a row are
// 8 contiguous bytes.
//
// Operand values of 2^60 or more (infinities among them): the terms of a split
// could overflow or form inf * 0 where the fp32 product does not, so a block that
// meets one sums its tile again in fp32 on the vector units.  So does one that meets
// a NaN in an MNMajor operand: values are split in pairs, whose remainders take 0
// times each other, and there the two belong to different outputs.  (In a KMajor
// operand they belong to the same one, which is NaN either way.)  Such a block takes
// the fp32 tiles through LDS (a train step of 6-256-256-10000 on 1024 rows with one
// NaN target column: 310 us, 197 without; 491 with operands read from memory per k).
#pragma once

#include "gemm_f32.h"

namespace ot {

typedef __bf16 x3_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 x3_bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 x3_bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t x3_u32x4 __attribute__((ext_vector_type(4)));
typedef float x3_f32x16 __attribute__((ext_vector_type(16)));

constexpr float kX3Huge = 1152921504606846976.f;   // 2^60

// Three bf16 terms of 8 fp32 values, packed two per word; big = max(big, |x|),
// which a NaN among x leaves as it was or (NAN_TOO) turns into NaN.
// The remainders come from v_dot2_f32_bf16, x + (-1) * term + 0 * other term,
// which reads a term in place (7 instructions a pair instead of 11 with the
// terms widened first) and is exact, since every remainder is representable.
template <bool NAN_TOO>
__device__ __forceinline__ void x3_split8(const float (&x)[8], x3_u32x4 (&t)[3], float& big) {
  // (-1, 0) and (0, -1); in registers, since as an inline constant -1.0 would not be a bf16 pair
  uint32_t c0 = 0x0000bf80u, c1 = 0xbf800000u;
  asm("" : "+s"(c0), "+s"(c1));
  const x3_bf16x2 first = __builtin_bit_cast(x3_bf16x2, c0), second = __builtin_bit_cast(x3_bf16x2, c1);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float a = x[2 * q], b = x[2 * q + 1];
    if constexpr (NAN_TOO)
      big = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(a), fabsf(b)), big);   // v_maximum3_f32
    else
      big = fmaxf(fmaxf(fabsf(a), fabsf(b)), big);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const x3_bf16x2 w = __builtin_convertvector(f32x2{a, b}, x3_bf16x2);
      t[p][q] = __builtin_bit_cast(uint32_t, w);
      if (p < 2) {
        a = __builtin_amdgcn_fdot2_f32_bf16(w, first, a, false);
        b = __builtin_amdgcn_fdot2_f32_bf16(w, second, b, false);
      }
    }
  }
}

// One operand of a block: global loads of a 16-deep k tile (T rows or columns of
// the operand from x0, `lim` in all), its split and LDS stores, and fragments.
template <Lay L, int T, bool PERM>
struct X3Operand {
  static constexpr int CHUNKS = 2 * T;                              // 8 values each
  static constexpr int N = (CHUNKS + 255) / 256;                    // chunks per thread
  static constexpr int PLANE = T * 32;
  static constexpr int BYTES = 3 * PLANE;
  static_assert(T % 32 == 0 && (L == Lay::KMajor || T == 32 || T == 64 || T == 128 || T == 256), "tile");
  const float* base;
  int64_t ld;
  int64_t off[N];
  int cnt[N];            // MNMajor: columns of the chunk inside the operand (<= 0: none)
  f32x4 v[N][2];

  static __device__ __forceinline__ int mn_swz(int kr) {
    return T >= 128 ? 4 * (kr & 3) : T == 64 ? 4 * ((kr >> 1) & 1) : 0;
  }
  // PERM: neighbouring threads store rows r and r + 32, kept 8 bank groups apart
  static __device__ __forceinline__ int row_at(int r) { return PERM ? (r * 32) ^ (((r >> 5) & 1) << 7) : r * 32; }
  static __device__ __forceinline__ bool mine(int i) { return CHUNKS % 256 == 0 || (int)threadIdx.x + i * 256 < CHUNKS; }

  __device__ __forceinline__ X3Operand(const float* p, int64_t ld_, int64_t x0, int64_t lim) : base(p), ld(ld_) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int ci = mine(i) ? threadIdx.x + i * 256 : 0;      // threads without a chunk load the first
      if constexpr (L == Lay::KMajor) {
        // rows past the operand read its last one; their results are not stored
        off[i] = min(x0 + ci / 2, lim - 1) * ld + 8 * (ci % 2);
        cnt[i] = 8;
      } else {
        const int64_t c = x0 + 8 * (ci % (T / 8));
        cnt[i] = (int)min((int64_t)8, lim - c);
        off[i] = (int64_t)(ci / (T / 8)) * ld + (c < lim ? c : 0);
      }
    }
  }
  // values [k0, k0 + 16) of the k range, a whole k tile of whole chunks
  __device__ __forceinline__ void load_whole(int64_t k0) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float* p = base + off[i] + (L == Lay::KMajor ? k0 : k0 * ld);
      v[i][0] = *reinterpret_cast<const f32x4*>(p);
      v[i][1] = *reinterpret_cast<const f32x4*>(p + 4);
    }
  }
  // the same for any tile of the k range that ends at kend (zeros past it)
  __device__ __forceinline__ void load(int64_t k0, int64_t kend) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int ci = threadIdx.x + i * 256;
      const float* p = base + off[i] + (L == Lay::KMajor ? k0 : k0 * ld);
      int n;                                              // leading values of the chunk that exist
      if constexpr (L == Lay::KMajor) n = (int)max((int64_t)0, min((int64_t)8, kend - k0 - 8 * (ci % 2)));
      else n = (k0 + ci / (T / 8) < kend) ? cnt[i] : 0;
      if (!mine(i)) n = 0;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f32x4 t = {0.f, 0.f, 0.f, 0.f};
        if (n >= 4 * h + 4) t = *reinterpret_cast<const f32x4*>(p + 4 * h);
        else
          for (int e = 0; e < 4; ++e)
            if (4 * h + e < n) t[e] = p[4 * h + e];
        v[i][h] = t;
      }
    }
  }
  __device__ __forceinline__ void store(unsigned char* lds, float& big) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (!mine(i)) continue;
      const int ci = threadIdx.x + i * 256;
      const float x[8] = {v[i][0][0], v[i][0][1], v[i][0][2], v[i][0][3],
                          v[i][1][0], v[i][1][1], v[i][1][2], v[i][1][3]};
      x3_u32x4 t[3];
      x3_split8<L == Lay::MNMajor>(x, t, big);
      int at;
      if constexpr (L == Lay::KMajor) {
        int r = ci / 2;
        if constexpr (PERM) r = (r & ~63) | ((r & 1) << 5) | ((r >> 1) & 31);
        at = row_at(r) + ((ci % 2) ^ ((r >> 3) & 1)) * 16;
      } else {
        const int kr = ci / (T / 8), ch = ci % (T / 8);
        at = kr * T * 2 + (ch ^ mn_swz(kr)) * 16;
      }
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<x3_u32x4*>(lds + p * PLANE + at) = t[p];
    }
  }
  // the values as they are, [16][T]
  __device__ __forceinline__ void store_f32(float* lds) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (!mine(i)) continue;
      const int ci = threadIdx.x + i * 256;
      if constexpr (L == Lay::KMajor) {
#pragma unroll
        for (int e = 0; e < 8; ++e) lds[(8 * (ci % 2) + e) * T + ci / 2] = v[i][e / 4][e % 4];
      } else {
        float* p = lds + ci / (T / 8) * T + 8 * (ci % (T / 8));
        *reinterpret_cast<f32x4*>(p) = v[i][0];
        *reinterpret_cast<f32x4*>(p + 4) = v[i][1];
      }
    }
  }
  // Operand of one MFMA: 32 LDS rows / columns from b0, this lane's 8 k values.
  static __device__ __forceinline__ x3_bf16x8 frag(const unsigned char* lds, int plane, int b0) {
    const int lane = threadIdx.x & 63;
    const unsigned char* p = lds + plane * PLANE;
    if constexpr (L == Lay::KMajor) {
      const int r = b0 + lane % 32, c = lane / 32;
      return *reinterpret_cast<const x3_bf16x8*>(p + row_at(r) + (c ^ ((r >> 3) & 1)) * 16);
    } else {
      typedef __attribute__((address_space(3))) x3_bf16x4 lds_bf16x4;
      const int c = lane % 16, q = lane / 16;
      const int col = b0 + 16 * (q & 1) + 4 * (c % 4);
      const int r0 = 8 * (q >> 1) + c / 4, r1 = r0 + 4;
      const int ch = col / 8, half = (col / 4) & 1;
      const x3_bf16x4 lo =
          __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + r0 * T * 2 + (ch ^ mn_swz(r0)) * 16 + half * 8));
      const x3_bf16x4 hi =
          __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + r1 * T * 2 + (ch ^ mn_swz(r1)) * 16 + half * 8));
      return x3_bf16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    }
  }
};

// Wavefronts per SIMD that the register budget is held to: two blocks of
// 128 x 128 or 256 columns share a CU (a third one spills its accumulators:
// 2.3 times the time), three of the smaller tiles.
constexpr int x3_waves(int wgn, int fm, int fn) { return (wgn == 4 || fm * fn >= 4) ? 2 : 3; }

// LDS-only barrier: __syncthreads() would also wait for the global loads that
// are meant to stay in flight.
__device__ __forceinline__ void x3_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int WGM, int WGN, int FM, int FN, Lay LA, Lay LB, Epi EPI, int ROLE = 0>
__global__ __launch_bounds__(256, x3_waves(WGN, FM, FN)) void gemm_f32x3_kernel(GemmArgs g) {
  static_assert(WGM * WGN == 4, "four wavefronts");
  constexpr int WM = 32 * FM, WN = 32 * FN, BM = WGM * WM, BN = WGN * WN;
  constexpr bool IL = (LB == Lay::KMajor) && FN == 2;     // interleaved output columns
  typedef X3Operand<LA, BM, false> OA;
  typedef X3Operand<LB, BN, IL> OB;
  constexpr int BUF = OA::BYTES + OB::BYTES;
  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * BUF];
  __shared__ int s_huge;
  __shared__ double s_red[4];
  __shared__ int32_t s_trow[EPI == Epi::Mse ? BM : 1];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wid % WGM, wn = wid / WGM;
  const int64_t tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  const int64_t lin = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  const int64_t l2 = xcd_remap(lin, (int64_t)gridDim.x * gridDim.y);
  const int64_t logical = l2 % gridDim.x, split = l2 / gridDim.x;
  int64_t tm, tn;
  if (tiles_m <= tiles_n) { tm = logical % tiles_m; tn = logical / tiles_m; }
  else { tn = logical % tiles_n; tm = logical / tiles_n; }
  const int64_t m0 = tm * BM, n0 = tn * BN;
  const int64_t kbeg = split * g.k_chunk;
  const int64_t kend = (kbeg + g.k_chunk < g.K) ? kbeg + g.k_chunk : g.K;
  const int64_t nk = (kend > kbeg) ? (kend - kbeg + 15) / 16 : 0;
  // k tiles that load_whole may read: every chunk of the block lies in its
  // operand's rows (rows past a KMajor operand are clamped; a chunk past an
  // MNMajor one must still lie in its padded row)
  const bool whole = (LA == Lay::KMajor || m0 + BM <= g.M || g.padded_a) &&
                     (LB == Lay::KMajor || n0 + BN <= g.N || g.padded_b);
  const int64_t nk_whole = whole && kend > kbeg ? (kend - kbeg) / 16 : 0;

  if (tid == 0) s_huge = 0;
  if constexpr (EPI == Epi::Mse) {
    if (g.target_rows && tid < BM) {
      const int64_t m = min(m0 + tid, g.M - 1);
      s_trow[tid] = (int32_t)min(max((int64_t)g.target_rows[m], (int64_t)0), g.target_rows_max);
    }
  }
  x3_barrier();

  OA oa(g.A, g.lda, m0, g.M);
  OB ob(g.B, g.ldb, n0, g.N);
  x3_f32x16 acc[FM][FN];
#pragma unroll
  for (int f = 0; f < FM; ++f)
#pragma unroll
    for (int h = 0; h < FN; ++h) acc[f][h] = x3_f32x16{};

  // row sums of an MNMajor A over k (the bias gradient), per chunk of this thread
  const bool do_rowsum = (LA == Lay::MNMajor) && g.rowsum != nullptr && tn == 0;
  float rs[OA::N][8];
#pragma unroll
  for (int i = 0; i < OA::N; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) rs[i][e] = 0.f;
  auto add_rowsum = [&] {
    if constexpr (LA == Lay::MNMajor) {
      if (do_rowsum) {
#pragma unroll
        for (int i = 0; i < OA::N; ++i)
#pragma unroll
          for (int e = 0; e < 8; ++e) rs[i][e] += oa.v[i][e / 4][e % 4];
      }
    }
  };
  auto load = [&](int64_t t) {
    if (t < nk_whole) {
      oa.load_whole(kbeg + 16 * t);
      ob.load_whole(kbeg + 16 * t);
    } else {
      oa.load(kbeg + 16 * t, kend);
      ob.load(kbeg + 16 * t, kend);
    }
  };
  x3_bf16x8 a[3][FM], b[3][FN];
  auto frags = [&](int buf) {
    const unsigned char* la = smem + buf * BUF;
    const unsigned char* lb = la + OA::BYTES;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
#pragma unroll
      for (int f = 0; f < FM; ++f) a[p][f] = OA::frag(la, p, WM * wm + 32 * f);
#pragma unroll
      for (int h = 0; h < FN; ++h) b[p][h] = OB::frag(lb, p, WN * wn + 32 * h);
    }
  };
  // The five smaller products of a step sum in accumulators of their own, so
  // that the large ones are rounded once per step as in a plain fp32 chain.
  x3_f32x16 low[FM][FN];
#pragma unroll
  for (int f = 0; f < FM; ++f)
#pragma unroll
    for (int h = 0; h < FN; ++h) low[f][h] = x3_f32x16{};
  auto mfmas = [&] {
    constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};   // smallest terms first
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int h = 0; h < FN; ++h) {
          x3_f32x16& d = q < 5 ? low[f][h] : acc[f][h];
          d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA[q]][f], b[PB[q]][h], d, 0, 0, 0);
        }
  };

  // output rows and columns of this lane
  const int64_t mw = m0 + WM * wm + 4 * (lane / 32), nw = n0 + WN * wn + (IL ? FN : 1) * (lane % 32);
  auto row_of = [&](int f, int r) { return mw + 32 * f + 8 * (r / 4) + r % 4; };
  auto col_of = [&](int h) { return nw + (IL ? h : 32 * h); };
  float big_a = 0.f, big_kb = 0.f;                       // largest |value| this thread has split, or NaN
  float& big_b = LA == LB ? big_a : big_kb;              // (the maximum of a KMajor operand would drop the NaN)
  auto store = [&](int buf) {
    add_rowsum();
    oa.store(smem + buf * BUF, big_a);
    ob.store(smem + buf * BUF + OA::BYTES, big_b);
  };
  int64_t t = 0;
  if (nk > 0) {
    load(0);
    store(0);
    if (nk > 1) load(1);
    x3_barrier();
  }
  // tiles whose successor's successor is whole: no branch inside
  for (; t + 2 < nk_whole; ++t) {
    frags((int)(t & 1));
    store((int)(t & 1) ^ 1);
    mfmas();
    oa.load_whole(kbeg + 16 * (t + 2));
    ob.load_whole(kbeg + 16 * (t + 2));
    x3_barrier();
  }
  for (; t < nk; ++t) {
    frags((int)(t & 1));
    mfmas();
    if (t + 1 < nk) {
      store((int)(t & 1) ^ 1);
      if (t + 2 < nk) load(t + 2);
    }
    x3_barrier();
  }
#pragma unroll
  for (int f = 0; f < FM; ++f)
#pragma unroll
    for (int h = 0; h < FN; ++h) acc[f][h] += low[f][h];

  if (!(big_a < kX3Huge && big_b < kX3Huge)) s_huge = 1;
  x3_barrier();
  if (__builtin_amdgcn_readfirstlane(s_huge)) {            // the same for the whole block
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
      for (int h = 0; h < FN; ++h) acc[f][h] = x3_f32x16{};
    float* fa = reinterpret_cast<float*>(smem);           // [16][BM], then [16][BN]
    float* fb = fa + 16 * BM;
    static_assert(64 * (BM + BN) <= 2 * BUF, "fp32 tile");
    for (int64_t q = 0; q < nk; ++q) {
      load(q);
      x3_barrier();                                       // the tile before has been read
      oa.store_f32(fa);
      ob.store_f32(fb);
      x3_barrier();
#pragma unroll 1
      for (int k = 0; k < 16; ++k) {
        float bk[FN];
#pragma unroll
        for (int h = 0; h < FN; ++h) bk[h] = fb[k * BN + WN * wn + (IL ? FN * (lane % 32) + h : 32 * h + lane % 32)];
#pragma unroll
        for (int f = 0; f < FM; ++f)
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) {
            const f32x4 ak = *reinterpret_cast<const f32x4*>(fa + k * BM + WM * wm + 32 * f + 8 * g4 + 4 * (lane / 32));
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
              for (int h = 0; h < FN; ++h) acc[f][h][4 * g4 + e] = fmaf(ak[e], bk[h], acc[f][h][4 * g4 + e]);
          }
      }
    }
    x3_barrier();
  }
  if constexpr (LA == Lay::MNMajor) {
    if (do_rowsum) {                                      // uniform over the block
      float* red = reinterpret_cast<float*>(smem);        // [16][BM]
#pragma unroll
      for (int i = 0; i < OA::N; ++i) {
        const int ci = tid + i * 256, kr = ci / (BM / 8), ch = ci % (BM / 8);
        if (OA::mine(i))
#pragma unroll
          for (int e = 0; e < 8; ++e) red[kr * BM + 8 * ch + e] = rs[i][e];
      }
      x3_barrier();
      if (tid < BM && m0 + tid < g.M) {
        float s = 0.f;
        for (int kr = 0; kr < 16; ++kr) s += red[kr * BM + tid];
        finish_rowsum<EPI>(g, split, m0 + tid, s);
      }
    }
  }

  // ---------------------------------------------------------------- epilogue
  float* Cb = g.C + (EPI == Epi::SplitK ? split * g.split_stride : 0);
  const bool full = col_of(FN - 1) < g.N;
  // this lane's FN values of a row starting at p (column 0 of the row)
  auto get = [&](const float* p, float* out) {
    if (IL && full) {
      const f32x2 t2 = *reinterpret_cast<const f32x2*>(p + nw);
      out[0] = t2[0];
      out[FN - 1] = t2[1];
    } else {
#pragma unroll
      for (int h = 0; h < FN; ++h) out[h] = col_of(h) < g.N ? p[col_of(h)] : 0.f;
    }
  };
  auto put = [&](float* p, const float* val) {
    if (IL && full) {
      *reinterpret_cast<f32x2*>(p + nw) = f32x2{val[0], val[FN - 1]};
    } else {
#pragma unroll
      for (int h = 0; h < FN; ++h)
        if (col_of(h) < g.N) p[col_of(h)] = val[h];
    }
  };
  float bias[FN];
  if constexpr (EPI == Epi::Bias || EPI == Epi::BiasRelu || EPI == Epi::Mse) get(g.bias, bias);
  if constexpr (EPI == Epi::Adam) {
    // The wavefront's gradients pass through its own part of LDS, 32 rows at a
    // time, so that a lane updates 4 consecutive parameters and a row is read
    // and written in runs of 128 FN bytes.  The loads of four passes are issued together.
    constexpr int EP = WN + 4, CG = WN / 4, RPP = 64 / CG, NP = 32 / RPP;
    static_assert(4 * 32 * EP * 4 <= 2 * BUF, "Adam staging");
    const AdamArgs ad = g.adam.resolved();
    float* ep = reinterpret_cast<float*>(smem) + wid * (32 * EP);
    const int cg = lane % CG, rl = lane / CG;
    const int64_t col = n0 + WN * wn + 4 * cg;
    const int cnt = (int)max((int64_t)0, min((int64_t)4, g.N - col));
    x3_barrier();                                          // the row sums have been read from LDS
#pragma unroll
    for (int f = 0; f < FM; ++f) {
#pragma unroll
      for (int h = 0; h < FN; ++h)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          ep[(8 * (r / 4) + 4 * (lane / 32) + r % 4) * EP + (IL ? FN * (lane % 32) + h : 32 * h + lane % 32)] =
              acc[f][h][r];
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // lanes read what other lanes of the wavefront wrote
      const int64_t mf = m0 + WM * wm + 32 * f;
#pragma unroll
      for (int i0 = 0; i0 < NP; i0 += 4) {
        if (cnt == 4) {
          f32x4 P[4], Mo[4], V[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int64_t o = min(mf + rl + RPP * (i0 + u), g.M - 1) * g.ldc + col;
            P[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(g.C + o));
            Mo[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(g.adam_m + o));
            V[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(g.adam_v + o));
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int rr = rl + RPP * (i0 + u);
            if (mf + rr >= g.M) continue;
            const int64_t o = (mf + rr) * g.ldc + col;
            adam4(P[u], *reinterpret_cast<const f32x4*>(ep + rr * EP + 4 * cg), Mo[u], V[u], ad);
            __builtin_nontemporal_store(P[u], reinterpret_cast<f32x4*>(g.C + o));
            __builtin_nontemporal_store(Mo[u], reinterpret_cast<f32x4*>(g.adam_m + o));
            __builtin_nontemporal_store(V[u], reinterpret_cast<f32x4*>(g.adam_v + o));
          }
        } else {
          for (int u = 0; u < 4; ++u) {
            const int rr = rl + RPP * (i0 + u);
            if (mf + rr >= g.M) continue;
            for (int c = 0; c < cnt; ++c) {
              const int64_t o = (mf + rr) * g.ldc + col + c;
              adam1(g.C[o], ep[rr * EP + 4 * cg + c], g.adam_m[o], g.adam_v[o], ad);
            }
          }
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    return;
  }
  float lsum = 0.f;
#pragma unroll
  for (int f = 0; f < FM; ++f) {
    // targets or masks of the fragment's 16 rows: all loads in flight together
    // (8 at a time: 1024 x 10000 x 256 in 74 us when 16 took 63)
    constexpr int RG = 16;
#pragma unroll
    for (int r0 = 0; r0 < 16; r0 += RG) {
      float pre[RG][FN];
      if constexpr (EPI == Epi::Mse || EPI == Epi::Mask) {
#pragma unroll
        for (int u = 0; u < RG; ++u) {
          const int64_t m = min(row_of(f, r0 + u), g.M - 1);
          if constexpr (EPI == Epi::Mse)
            get(g.target + (g.target_rows ? (int64_t)s_trow[m - m0] : m) * g.ldt, pre[u]);
          else get(g.mask + m * g.ldmask, pre[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < RG; ++u) {
        const int64_t m = row_of(f, r0 + u);
        if (m >= g.M) continue;
        float val[FN];
#pragma unroll
        for (int h = 0; h < FN; ++h) {
          float x = acc[f][h][r0 + u];
          if constexpr (EPI == Epi::Bias || EPI == Epi::BiasRelu || EPI == Epi::Mse) x += bias[h];
          if constexpr (EPI == Epi::BiasRelu) x = x > 0.f ? x : 0.f;
          if constexpr (EPI == Epi::Mask) x = pre[u][h] > 0.f ? x : 0.f;
          if constexpr (EPI == Epi::Mse) {
            const float d = col_of(h) < g.N ? x - pre[u][h] : 0.f;
            lsum += d * d;
            x = g.scale * d;
          }
          val[h] = x;
        }
        put(Cb + m * g.ldc, val);
      }
    }
  }
  if constexpr (EPI == Epi::Mse) {
    const double ls = warp_sum((double)lsum);
    if (lane == 0) s_red[wid] = ls;
    x3_barrier();
    if (tid == 0) {
      g.loss_partials[blockIdx.y * gridDim.x + blockIdx.x] = ((s_red[0] + s_red[1]) + s_red[2]) + s_red[3];
      if (g.step_now && blockIdx.x == 0) *g.step_now += 1;
    }
  }
}

template <int WGM, int WGN, int FM, int FN, Lay LA, Lay LB, Epi EPI, int ROLE = 0>
hipError_t launch_gemm_f32x3(const GemmArgs& g, int64_t splits, hipStream_t stream, hipEvent_t t0 = nullptr,
                             hipEvent_t t1 = nullptr) {
  constexpr int BM = 32 * FM * WGM, BN = 32 * FN * WGN;
  const int64_t tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  hipExtLaunchKernelGGL((gemm_f32x3_kernel<WGM, WGN, FM, FN, LA, LB, EPI, ROLE>), dim3((unsigned)tiles, (unsigned)splits),
                        dim3(256), 0, stream, t0, t1, 0, g);
  return hipGetLastError();
}

}  // namespace ot
