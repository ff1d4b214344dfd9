// Dense layers of fp32 models on the bf16 matrix cores.
#include <cmath>

#include "device.h"
#include "launch.h"

namespace {

// Two fp32 values of at least 2^-110 (or 0) as the exact sums of three bf16
// values each (h + m + l; the first value in the low halves): a bf16 holds 8
// significant bits and each remainder is exact in fp32, so three hold all 24
// (under 2^-110 the last part would fall below the smallest bf16, 2^-133).
__device__ __forceinline__ void split3(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = pack2_rne(a, b);
  const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
  m = pack2_rne(ra, rb);
  l = pack2_rne(ra - __uint_as_float(m << 16), rb - __uint_as_float(m & 0xffff0000u));
}

// Every LDS operation of this wave done, then all waves of the workgroup meet
// (global loads into registers stay in flight, unlike with __syncthreads).
__device__ __forceinline__ void lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The rows of X gathered instead of read at a fixed stride: row r starts at
// element src[r * stride] of X (len elements). A row outside it (padding, -1)
// reads as zeros; one that starts inside but ends past the end also sets *err
// (when given).
struct GatherArgs {
  const int64_t* src;
  int stride;
  int64_t len;
  int* err;
};

__device__ float k_zeros[64];  // one k-step of a row of zeros

// Y = act(X W^T + b) with fp32 X, W, b and Y, on the bf16 matrix cores (fp32
// MFMA peaks at 157 TFLOP/s, bf16 at 2500): every operand is the exact sum of
// three bf16 parts, and a product is the sum of its six partial products down
// to 2^-16 of it, each exact in fp32, accumulated in fp32 (three-way splitting
// as published for emulating single precision on bf16 units, Henry et al. 2019).
// The three partial products left out are below 2^-26 of the product, under an
// fp32 rounding.
//
// X is scaled by 2^40 before it is split, so that every fp32 value down to the
// smallest, 2^-149, is the sum of its parts, and W by a power of two that the
// model loader picks for its smallest weight (1 unless one is under 2^-110);
// `unscale` takes both out of the sum. A sum that overflows for it (2^88 and
// more, without such weights) is one of the non-finite ones below.
//
// The products of the first parts have an accumulator of their own, and the
// five smaller ones another (below 2^-7 of it, so that its roundings do not
// count); the two meet at the end. The first one is then rounded once for
// every 8 k values with a product that is not zero, where the fp32 MFMA rounds
// once for each such product: on no input has the sum more roundings than the
// fp32 MFMA's. With one accumulator for all six it had 12 for 16 k values,
// more than the fp32 MFMA where half of X is zeros, as after a ReLU. Error
// against 64 bits over the result's norm at K = 1024, of the fp32 MFMA, of one
// accumulator and of two: normal inputs 5.7e-7, 4.9e-7, 1.8e-7; half of them
// zeros 4.1e-7, 4.7e-7, 1.4e-7; nine of ten zeros 1.8e-7 and 0.6e-7 (the first
// and the last).
//
// W comes split (rb_split_f32_weights): per 32 rows and 16 k values the three
// parts in the order of a wave's fragment, so a fragment is one coalesced load
// from L2 into registers, RBUF - 1 sub-steps of 16 k values ahead. X is split
// once per workgroup and k-step (16 KS values) on its way from registers to one
// of two LDS stages; there a part of 32 rows x 16 k values takes ABLK 16-byte
// units, its second k half 40 units after the first (each part's 8-byte writes
// and 16-byte fragment reads then spread over all banks).
//
// PIPE: with few waves per SIMD the order is fixed by hand: each MFMA is
// followed by its share of the k-step's other work, and the next fragments
// are read before they are needed (512 x 1024 x 1024: 17 us, against 30 us in
// program order). Otherwise four waves per SIMD overlap each other's phases
// (64 x 256 tiles; 262144 x 512 x 256: 423 us, 384 us with 128 x 256 tiles and
// one accumulator; two accumulators leave no registers for four waves of 128
// rows, and 128 x 256 tiles of two waves per SIMD take 422 to 434 us, 64 x 256
// with the six products summed from zero and added by vector adds 410 to 420 us
// but 3 to 8% more for launches of few rows).
//
// Every tile shape accumulates an output element in the same k order with the
// same instructions, so results depend neither on it nor on which rows share
// a tile.
template <int BM, int BN, int WM, int WN, int KS, int RBUF, bool PIPE, int ACT>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64, PIPE ? 2 : 4) void k_gemm_f32_split(
    const float* __restrict__ X, int ldx, GatherArgs ga, const u32x4_t* __restrict__ Wp,
    const float* __restrict__ bias, float* __restrict__ Y, int ldy, int M, int N, int K, float unscale,
    int xcd_order, const rb_k_row* __restrict__ skip_rows, int skip_T, OutMap om) {
  constexpr int NT = (BM / WM) * (BN / WN) * 64;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int BK = 16 * KS;           // k values per k-step
  constexpr int LA = BM * 4 * KS / NT;  // groups of 4 values each thread splits per k-step
  constexpr int ABLK = 72;
  static_assert(LA * NT == BM * 4 * KS && KS % RBUF == 0 && KS % 2 == 0 && BK <= 64, "groups cover the tile");
  __shared__ u32x4_t sA[2][KS * (BM / 32) * 3 * ABLK];
  constexpr uint32_t STAGE = sizeof(sA[0]);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wid / (BN / WN), wn = wid % (BN / WN);
  const int tiles_n = N / BN;
  const int tile = xcd_order ? xcd_tile(blockIdx.x, gridDim.x) : blockIdx.x;
  const int m0 = tile / tiles_n * BM, n0 = tile % tiles_n * BN;
  int64_t live = M;  // rows from here on hold padding tokens
  if (skip_rows) {   // uniform per workgroup
    const int e = m0 / skip_T;
    const rb_k_row rw = skip_rows[e];
    if (rw.src < 0 || m0 - e * skip_T >= rw.aux) return;
    live = e * (int64_t)skip_T + rw.aux;
  }
  // start of X's row r (rows past M: the last one, never stored), or null for a row of zeros
  auto row_ptr = [&](int r) -> const float* {
    r = min(r, M - 1);
    if (!ga.src) return X + (int64_t)r * ldx;
    const int64_t s = ga.src[(int64_t)r * ga.stride];
    const bool in = s >= 0 && s <= ga.len - K;
    if (s >= 0 && !in && ga.err) *ga.err = 1;
    return in ? X + s : nullptr;
  };
  // group i of thread t: with u = t + i NT, values 4 (u % 4) .. + 3 of the 16 k
  // values u / (4 BM) of row u / 4 % BM; rows may start at any multiple of 4 bytes
  typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
  const float* pa[LA];
  int ma[LA];  // mask of the k offset (0 for a row of zeros)
  uint32_t wa[LA];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int u = tid + i * NT, q = u & 3, r = (u >> 2) % BM, ks = u / (4 * BM);
    const float* p = row_ptr(m0 + r);
    ma[i] = p ? -1 : 0;
    pa[i] = (p ? p : k_zeros) + ks * 16 + q * 4;
    wa[i] = ((ks * (BM / 32) + (r >> 5)) * 3 * ABLK + (q >> 1) * 40 + (r & 31)) * 16 + (q & 1) * 8;
  }
  f32x4_t ra[LA];
  const int nk = K / BK, nsub = K / 16;
  auto load_a = [&](auto ic_, int kt) {  // k-steps past the end: the last one again, never used
    constexpr int i = decltype(ic_)::value;
    ra[i] = *(const f32x4_any*)(pa[i] + ((min(kt, nk - 1) * BK) & ma[i]));
  };
  // half hc (two values) of group i split; with the second half, its parts go
  // to the LDS stage at byte offset st
  u32x2_t sh, sm, sl;
  auto split_half = [&](uint32_t st, auto ic_, auto hc) {
    constexpr int i = decltype(ic_)::value, h = decltype(hc)::value;
    uint32_t a, b, c;
    split3(ra[i][2 * h] * 0x1p40f, ra[i][2 * h + 1] * 0x1p40f, a, b, c);
    sh[h] = a;
    sm[h] = b;
    sl[h] = c;
    if constexpr (h == 1) {
      unsigned char* base = (unsigned char*)sA + (wa[i] + st);
      *(u32x2_t*)base = sh;
      *(u32x2_t*)(base + ABLK * 16) = sm;
      *(u32x2_t*)(base + 2 * ABLK * 16) = sl;
    }
  };
  // W's fragments of one sub-step, q-th load: part 2 - q / TN of column block q % TN
  u32x4_t fb[RBUF][3][TN];
  const u32x4_t* wbase = Wp + (int64_t)((n0 + wn * WN) / 32) * nsub * 192 + lane;
  auto load_b = [&](auto bufc, auto qc, int sub) {
    constexpr int bf = decltype(bufc)::value, q = decltype(qc)::value, p = 2 - q / TN, j = q % TN;
    fb[bf][p][j] = wbase[((int64_t)j * nsub + min(sub, nsub - 1)) * 192 + p * 64];
  };
  // X's fragments of sub-step ks of the stage at st, q-th read: part 2 - q / TM
  // of row block q % TM (lane l holds row l % 32, k values 8 (l / 32) .. + 7)
  u32x4_t fa[PIPE ? 2 : 1][3][TM];
  const uint32_t ra0 = (uint32_t)(wm * TM * 3 * ABLK + (lane >> 5) * 40 + (lane & 31)) * 16;
  auto read_a = [&](uint32_t st, auto ksc, auto qc, auto bufc) {
    constexpr int ks = decltype(ksc)::value, q = decltype(qc)::value, p = 2 - q / TM, i = q % TM;
    fa[decltype(bufc)::value][p][i] =
        *(const u32x4_t*)((const unsigned char*)sA + (ra0 + st) + ((ks * (BM / 32) + i) * 3 + p) * ABLK * 16);
  };
  floatx16_t acc[TM][TN], low[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = low[i][j][r] = 0.f;
  constexpr int NM = TM * TN, NU = 6 * NM;  // MFMAs per sub-step
  constexpr int NS = KS * NU;               // MFMAs per k-step
  constexpr int UB = NS - NU / 2;           // of them before the barrier (PIPE)
  // the parts of the six partial products, smallest first; the last one's sum is acc
  constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
  auto mfma = [&](auto abufc, auto bbufc, auto vc) {
    constexpr int v = decltype(vc)::value, p = v / NM, m = v % NM;
    floatx16_t& sum = (p < 5 ? low : acc)[m / TN][m % TN];
    sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
        __builtin_bit_cast(bf16x8_t, fa[decltype(abufc)::value][PA[p]][m / TN]),
        __builtin_bit_cast(bf16x8_t, fb[decltype(bbufc)::value][PB[p]][m % TN]), sum, 0, 0, 0);
  };
  static_for<LA>([&](auto c) { load_a(c, 0); });
  static_for<RBUF - 1>([&](auto sc) { static_for<3 * TN>([&](auto qc) { load_b(sc, qc, decltype(sc)::value); }); });
  static_for<LA>([&](auto c) {
    split_half(0, c, ic<0>{});
    split_half(0, c, ic<1>{});
    load_a(c, 1);
  });
  lds_sync();
  uint32_t st = 0;
  if constexpr (PIPE) static_for<3 * TM>([&](auto qc) { read_a(0, ic<0>{}, qc, ic<0>{}); });
  for (int kt = 0; kt < nk; ++kt) {
    const uint32_t nst = STAGE - st;
    if constexpr (PIPE) {
      static_for<NS>([&](auto uc) {
        constexpr int u = decltype(uc)::value, ks = u / NU, v = u % NU;
        // the next stage is whole, and this one's fragments have all been read
        if constexpr (u == UB) lds_sync();
        mfma(ic<ks & 1>{}, ic<ks % RBUF>{}, ic<v>{});
        __builtin_amdgcn_sched_barrier(0);
        static_for<3 * TM>([&](auto qc) {
          constexpr int q = decltype(qc)::value;
          if constexpr (ks + 1 < KS) {
            if constexpr (q * NU / (3 * TM) == v) read_a(st, ic<ks + 1>{}, qc, ic<(ks + 1) & 1>{});
          } else {
            if constexpr (UB + q * (NS - UB) / (3 * TM) == u) read_a(nst, ic<0>{}, qc, ic<0>{});
          }
        });
        static_for<3 * TN>([&](auto qc) {
          constexpr int q = decltype(qc)::value;
          if constexpr (q * NU / (3 * TN) == v) load_b(ic<(ks + RBUF - 1) % RBUF>{}, qc, kt * KS + ks + RBUF - 1);
        });
        static_for<2 * LA>([&](auto qc) {
          constexpr int q = decltype(qc)::value, i = q / 2;
          if constexpr (q * (UB - 1) / (2 * LA) == u) {
            split_half(nst, ic<i>{}, ic<q & 1>{});
            if constexpr (q & 1) load_a(ic<i>{}, kt + 2);
          }
        });
        __builtin_amdgcn_sched_barrier(0);
      });
    } else {
      static_for<KS>([&](auto ksc) {
        constexpr int ks = decltype(ksc)::value;
        static_for<3 * TN>([&](auto qc) { load_b(ic<(ks + RBUF - 1) % RBUF>{}, qc, kt * KS + ks + RBUF - 1); });
        static_for<3 * TM>([&](auto qc) { read_a(st, ksc, qc, ic<0>{}); });
        static_for<NU>([&](auto vc) { mfma(ic<0>{}, ic<ks % RBUF>{}, vc); });
        if constexpr (ks == 0)
          static_for<LA>([&](auto c) {
            split_half(nst, c, ic<0>{});
            split_half(nst, c, ic<1>{});
            load_a(c, kt + 2);
          });
      });
      lds_sync();
    }
    st = nst;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] += low[i][j];
  // Infinities, NaN and values that the scaling takes past the end of the fp32
  // range: an operand's split then has infinite or NaN parts, which make every
  // sum they enter non-finite. Those elements (and no others, so that a row's result does not
  // depend on its neighbours) are computed again with fp32 operands.
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int rl = m0 + wm * WM + i * 32;
      bool bad = false;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        bad |= !isfinite(acc[i][j][r]) && rl + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3) < live;
      if (__any(bad)) {
        floatx16_t z;
#pragma unroll
        for (int r = 0; r < 16; ++r) z[r] = 0.f;
        const float* xr = row_ptr(rl + (lane & 31));
        const uint16_t* wr = (const uint16_t*)(Wp + (int64_t)((n0 + wn * WN) / 32 + j) * nsub * 192);
        for (int k0 = 0; k0 < K; k0 += 2) {
          const int k = k0 + (lane >> 5);  // lane l: row l % 32, k value l / 32
          const uint16_t* e = wr + (k >> 4) * 1536 + ((((k >> 3) & 1) << 5) + (lane & 31)) * 8 + (k & 7);
          float w = bf2f(e[0]);
          if (isfinite(w)) w += bf2f(e[512]) + bf2f(e[1024]);  // exact; a non-finite w has itself as its first part
          w *= unscale * 0x1p40f;                              // W's part of the scale
          z = __builtin_amdgcn_mfma_f32_32x32x2f32(xr ? xr[k] : 0.f, w, z, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = isfinite(acc[i][j][r]) ? acc[i][j][r] * unscale : z[r];
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] *= unscale;
      }
    }
  // the store, as in gemm_mfma's epilogue: each group of four registers (four
  // consecutive rows) transposed across the lanes of a quad
  int64_t ro[TM][4];
  if (om.rows) {  // uniform; the output offsets of this lane's rows, loaded at once
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int r = m0 + wm * WM + i * 32 + 8 * g + 4 * (lane >> 5) + (lane & 3);
        ro[i][g] = r < M ? om.rows[r].out : -1;
      }
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const float bb = bias[n0 + wn * WN + j * 32 + (lane & 31)];
    const int colq = n0 + wn * WN + j * 32 + (lane & 28);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float q[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) q[k] = act_fn<ACT>(acc[i][j][4 * g + k] + bb);
        quad_transpose4(q, lane);
        const int row = m0 + wm * WM + i * 32 + 8 * g + 4 * (lane >> 5) + (lane & 3);
        const f32x4_t v = {q[0], q[1], q[2], q[3]};
        if (!om.rows) {
          if (row < M) __builtin_nontemporal_store(v, (f32x4_t*)(Y + (int64_t)row * ldy + colq));
        } else if (ro[i][g] >= 0) {
          float* dst = om.out + ro[i][g] + colq;
          if (colq + 3 < om.d_out && ((uintptr_t)dst & 15) == 0) {
            __builtin_nontemporal_store(v, (f32x4_t*)dst);
          } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
              if (colq + k < om.d_out) dst[k] = q[k];
          }
        }
      }
  }
}

// W [N, K] times scale as three bf16 parts per element that sum to it exactly
// (a finite element's first part is not rounded up to infinity, a non-finite one
// is its own first part), [Np, Kp] zero padded: per 32 rows and 16 k values the
// parts one after another, each in the order of a wave's 32 x 16 fragment. A
// thread splits eight k values of a row, consecutive threads consecutive rows
// (whole lines stored; 4096 x 4096 at load: 114 ms with the split on the host).
__global__ __launch_bounds__(256) void k_split_weights(const float* __restrict__ W, int N, int K, int Np, int Kp,
                                                       float scale, u32x4_t* __restrict__ Wp) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // unit i % 64 of 16 k values of 32 rows
  if (i >= (int64_t)Np * Kp / 8) return;
  const int64_t block = i >> 6;
  const int u = (int)(i & 63), nsub = Kp / 16;
  const int j = (int)(block / nsub) * 32 + (u & 31), k0 = (int)(block % nsub) * 16 + (u >> 5) * 8;
  uint32_t part[3][8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    float r = j < N && k0 + k < K ? W[(int64_t)j * K + k0 + k] * scale : 0.f;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      uint32_t v = f2bf(r);
      if ((v & 0x7fff) == 0x7f80 && isfinite(r)) --v;
      part[p][k] = v;
      r = (v & 0x7f80) == 0x7f80 ? 0.f : r - bf2f(v);
    }
  }
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const uint32_t* h = part[p];
    Wp[block * 192 + p * 64 + u] =
        (u32x4_t){h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
  }
}

}  // namespace

// Runtime support (not part of the C ABI): split weights (above) from fp32 ones
// in device memory.
rb_status rb_split_f32_weights(hipStream_t s, const float* W, int N, int K, int Np, int Kp, float scale, void* Wp) {
  if (N < 1 || K < 1 || Np < N || Kp < K || Np % 32 || Kp % 16 || !W || !Wp) return RB_EINVAL;
  hipLaunchKernelGGL(k_split_weights, dim3((unsigned)(((int64_t)Np * Kp / 8 + 255) / 256)), dim3(256), 0, s, W, N, K, Np,
                     Kp, scale, (u32x4_t*)Wp);
  return launch_status();
}

// Runtime support (not part of the C ABI): one layer of an fp32 model on
// weights split by the model loader (three bf16 parts per element, in fragment
// order). X's rows are read at stride ldx, or gathered: row r from element
// src[r * src_stride] of X (src_len elements; K of them per row). The output
// goes to Y, or through the row map to out (out_rows given). skip_rows as in
// rb_k_gemm_f32. K and N are multiples of 64. Wp holds W times 2^w_exp (0..39).
rb_status rb_gemm_f32_split(hipStream_t s, const float* X, int ldx, const int64_t* src, int src_stride,
                            int64_t src_len, int* err, const void* Wp, int w_exp, const float* b, float* Y, int ldy,
                            int M, int N, int K, int act, const rb_k_row* skip_rows, int skip_T, const rb_k_row* out_rows, int d_out,
                            float* out) {
  if (M < 0 || N <= 0 || K <= 0 || N % 64 || K % 64 || !X || !Wp || !b || (!out_rows && (!Y || ldy < N)))
    return RB_EINVAL;
  if (act != RB_ACT_NONE && act != RB_ACT_RELU && act != RB_ACT_SIGMOID) return RB_EINVAL;
  if (skip_rows && (skip_T <= 0 || skip_T % 64)) return RB_EINVAL;
  if (M == 0) return RB_OK;
  const GatherArgs ga{src, src_stride, src_len, err};
  const OutMap om{out_rows, out, d_out};
  const float unscale = std::ldexp(1.f, -40 - w_exp);
  // XCD-contiguous tile order when all of W fits in one XCD's L2 (each XCD
  // then reads its X rows once), plain order otherwise
  const int xcd = (int64_t)N * K * 6 <= (4 << 20);
#define RB_S(BM, BN, WM, WN, KS, RBUF, PIPE, A)                                                                     \
  hipLaunchKernelGGL((k_gemm_f32_split<BM, BN, WM, WN, KS, RBUF, PIPE, A>),                                         \
                     dim3((unsigned)((M + BM - 1) / BM) * (N / BN)), dim3((BM / WM) * (BN / WN) * 64), 0, s, X, ldx, ga, \
                     (const u32x4_t*)Wp, b, Y, ldy, M, N, K, unscale, xcd, skip_rows, skip_T, om)
#define RB_L(...)                                          \
  do {                                                     \
    if (act == RB_ACT_RELU) RB_S(__VA_ARGS__, RB_ACT_RELU); \
    else if (act == RB_ACT_SIGMOID) RB_S(__VA_ARGS__, RB_ACT_SIGMOID); \
    else RB_S(__VA_ARGS__, RB_ACT_NONE);                   \
  } while (0)
  // The largest tile that fills the chip: 64 x 256 (8 waves, four a SIMD) with
  // four tiles for every compute unit, 64 x 128 (4 waves) with one, else
  // 32 x 64 (2 waves; 512 x 1024 x 1024: 17 us, against 22 us with 64 x 128).
  const int64_t cus = device_cus();
  if (!skip_rows && N % 256 == 0 && (int64_t)((M + 63) / 64) * (N / 256) >= 4 * cus)
    RB_L(64, 256, 64, 32, 2, 2, false);
  else if (N % 128 == 0 && (int64_t)((M + 63) / 64) * (N / 128) >= cus)
    RB_L(64, 128, 64, 32, 4, 4, true);
  else
    RB_L(32, 64, 32, 32, 4, 4, true);
#undef RB_L
#undef RB_S
  return launch_status();
}
