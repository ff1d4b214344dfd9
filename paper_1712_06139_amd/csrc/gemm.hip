// Dense layers on matrix cores: bf16 operands (a model's layers, and a last
// hidden layer fused with its head), and fp32 operands on the fp32 MFMA (the
// C ABI's fp32 entry points; an fp32 model's layers run in gemm_f32_split.hip).
#include "device.h"

namespace {

// Y = act(X W^T + b): X [M, K] and W [N, K] of element type TI (bf16 or
// fp32), K contiguous; fp32 accumulation with v_mfma_f32_16x16x32_bf16 or
// v_mfma_f32_32x32x2f32.
//
// Workgroup tile BM x BN, k-step of RB bytes per row (64 or 128: 16 or 32
// fp32; bf16 outputs take 128, 64 bf16), NT/64 waves each owning a WM x WN sub-tile
// ((WM/T) x (WN/T) accumulators; T = 16 bf16, 32 fp32). Operand tiles go straight from global
// memory into a ring of S >= 2 LDS stages (global_load_lds: each wave load
// instruction fills 1 KB of consecutive LDS rows; no register staging).
// K-step kt reads stage kt % S while the stage of k-step kt - 1 is refilled
// with k-step kt - 1 + S, its loads spread one every few MFMAs over the step
// (over its first half when S = 2, where that refill is the next k-step):
// issued back to back they stall the wave on the texture path with no MFMA in
// flight. A sub-step covers 32 bf16 or 8 fp32 k values of every row and its MFMAs have the next sub-step's fragment reads between them. In the
// last sub-step, after half of its MFMAs (three quarters with S = 2), the wave
// waits for its loads of the next k-step and for its LDS reads, and all waves
// meet at one barrier: the next stage has landed and nobody reads the current
// one again. The rest of the sub-step then runs with the next k-step's first
// fragment reads between the MFMAs. The order of MFMAs, LDS reads and loads
// within a step is fixed with scheduling barriers.
//
// A fragment is 16 bytes of one row: lane l holds row l % T and chunk l / T of
// the sub-step's. bf16: one 16x16x32 MFMA per accumulator and sub-step. It takes
// less power: with random operands in registers the chip sustains 2080 TFLOP/s
// of 16x16x32 against 1740 to 1800 of 32x32x16 (zeros: 2450 with either); the
// results have the same bits. 8192 x 1024 x 1728
// 28.4 -> 25.3 us, 32768 x 1024 x 1728 117 -> 96, 32768 x 512 x 1024 35 -> 32,
// 4096 x 4096 x 8192 202 -> 189, 65536 x 8192 x 4096 3290 either way. fp32:
// chunk c holds k = 4c .. 4c + 3, and MFMA t (t = 0..3) of the sub-step takes
// dword t, so it adds the products of k = 8 kk + t (lanes 0..31) and k = 8 kk + 4
// + t (lanes 32..63); the MFMAs of a sub-step run t-major over the accumulators,
// so two MFMAs into one accumulator are NM instructions apart.
//
// LDS rows hold RB/16 16-byte chunks; chunk c of row r sits at chunk
// c ^ ((r / (16 / (RB/16))) % (RB/16)), so the 16 rows one fragment read
// serves per LDS cycle hit 16 distinct bank groups (64 banks). For bf16
// outputs the column blocks of a wave come in pairs that take alternate groups of four of 32
// rows of W, so that a lane ends up with eight consecutive output columns, and
// W's rows have a permutation to match (swz_b).
//
// Every tile shape, k-step, stage count and tile order accumulates each output
// element in the same k order with the same instructions, so results do not
// depend on them, nor on which rows share a tile.
//
// skip_rows (sequence layout, slot e owning rows [e skip_T, (e + 1) skip_T),
// skip_T a multiple of BM): a workgroup whose rows are all padding tokens
// (at or past its slot's length, or in a padding slot) returns at once.
constexpr int G16_KALIGN = 64;  // K multiple the bf16 entry point accepts
constexpr int G32_KALIGN = 32;  // K multiple the fp32 entry point accepts
constexpr int G32_BM = 64;      // fp32 tile height (the padding-token skip granularity)

template <typename TI, int BM, int BN, int WM, int WN, int NT, int RB, int S, int ACT, bool OUT_F32,
          bool PERSIST, int HEAD = -1>
__device__ __forceinline__ void gemm_mfma(const TI* __restrict__ X, int ldx, const TI* __restrict__ W, int ldw,
                                          const float* __restrict__ bias, void* __restrict__ Y, int ldy, int M,
                                          int N, int K, int xcd_order, const rb_k_row* __restrict__ skip_rows, int skip_T,
                                          const HeadArgs ha = HeadArgs{}, const OutMap om = OutMap{}) {
  constexpr bool F32 = sizeof(TI) == 4;
  constexpr int ES = sizeof(TI);  // bytes per element
  constexpr int BK = RB / ES;     // k values per k-step
  constexpr int NW = NT / 64;
  static_assert((BM / WM) * (BN / WN) == NW, "one wave per sub-tile");
  static_assert(RB == 64 || RB == 128, "k-step of 64 or 128 bytes per row");
  static_assert(S >= 2 && S <= 8, "2..8 stages");
  constexpr int CPR = RB / 16;   // 16-byte chunks per LDS row
  constexpr int RPI = 64 / CPR;  // rows filled per wave load instruction
  constexpr int SWZ = 16 / CPR;  // rows sharing one swizzle pattern
  constexpr int EPC = 16 / ES;   // elements per chunk
  constexpr int T = F32 ? 32 : 16;       // rows and columns of one MFMA
  constexpr int NREG = T * T / 64;       // its accumulator registers
  constexpr int TM = WM / T, TN = WN / T;
  constexpr bool PAIR = !F32 && !OUT_F32;  // column blocks stored in pairs
  static_assert(F32 || TN % 2 == 0, "column blocks are stored in pairs");
  static_assert(!PAIR || CPR == 8, "the paired blocks' swizzle permutes eight chunks");
  typedef typename std::conditional<F32, floatx16_t, floatx4_t>::type acc_t;
  constexpr int SA = BM / RPI / NW, SB = BN / RPI / NW;  // load instructions per wave per stage
  static_assert(SA * NW * RPI == BM && SB * NW * RPI == BN, "loads cover the tile");
  constexpr int OPS = SA + SB;
  constexpr int CPS = 64 / T;    // 16-byte chunks of a row per sub-step (lane l holds chunk l / T of row l % T)
  constexpr int KK = CPR / CPS;  // MFMA sub-steps per k-step
  constexpr int NM = TM * TN;    // accumulators
  constexpr int MPF = F32 ? 4 : 1;  // MFMAs per accumulator and sub-step
  constexpr int NU = NM * MPF;   // MFMAs per sub-step
  constexpr int NR = TM + TN;    // fragment reads per sub-step
  // the last sub-step's MFMAs before the barrier: half of them, three quarters
  // with two stages (more time for the loads of the next k-step to land)
  constexpr int UB = S == 2 ? NU * 3 / 4 : NU / 2;
  constexpr int PRE = (KK - 1) * NU + UB;  // MFMAs of a step before its barrier
  // MFMA slots the refill loads are spread over: with two stages the stage
  // refilled during a step is the one the next step reads, so its loads go in
  // the first half of the step to land before the barrier
  constexpr int LPOS = S == 2 ? PRE / 2 : PRE;
  // fragment read slot -> fragment (A fragments q < TM, then B). With two
  // stages (bf16) in the order the next sub-step's MFMAs consume them (A0, B0
  // .. B(TN-1), A1 .. A(TM-1)), so the fragment needed first is read first;
  // otherwise A0 .. A(TM-1), B0 .. B(TN-1).
  auto qmap = [](auto sc) {
    constexpr int q = decltype(sc)::value;
    if constexpr (S != 2 || F32 || q == 0)
      return ic<q>{};
    else if constexpr (q <= TN)
      return ic<TM + q - 1>{};
    else
      return ic<q - TN>{};
  };
  __shared__ u32x4_t sA[S][BM * CPR];
  __shared__ u32x4_t sB[S][BN * CPR];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wid / (BN / WN), wn = wid % (BN / WN);
  const int tiles_n = N / BN;
  const int ntiles = ((M + BM - 1) / BM) * tiles_n;
  // v: this workgroup's index in the tile sequence (blockIdx.x, then + gridDim.x
  // per tile when persistent; gridDim.x is a multiple of 8, so v % 8 stays the
  // XCD the workgroup runs on)
  int v = blockIdx.x;
  auto tile_origin = [&](int vv, int& m0_, int& n0_) {
    const int tile = xcd_order ? xcd_tile(vv, ntiles) : vv;
    const int bm = tile / tiles_n;
    m0_ = bm * BM;
    n0_ = (tile - bm * tiles_n) * BN;
  };
  int m0, n0;
  tile_origin(v, m0, n0);
  if (skip_rows) {  // uniform per workgroup
    const int e = m0 / skip_T;
    const rb_k_row rw = skip_rows[e];
    if (rw.src < 0 || m0 - e * skip_T >= rw.aux) return;
  }

  // chunk c of row r sits at chunk c ^ swz(r); the column blocks of a pair take
  // alternate groups of 4 rows of W's 32, so their swizzle differs
  auto swz_a = [](int r) { return (r / SWZ) % CPR; };
  auto swz_b = [](int r) {
    if constexpr (!PAIR) return (r / SWZ) % CPR;
    else return ((r >> 1) & 1) | (((r >> 3) & 3) << 1);
  };
  // the row of W's tile that row x of a wave's column block j is
  auto b_row = [&](int j, int x) {
    if constexpr (!PAIR) return wn * WN + j * T + x;
    else return wn * WN + (j >> 1) * 32 + (x >> 2) * 8 + (j & 1) * 4 + (x & 3);
  };
  // lane l of a load instruction fills LDS row l / CPR (of its RPI), chunk l % CPR
  const int lr = lane / CPR, lc = lane % CPR;
  // byte offsets from the tile's first row (buffer resources based there; the
  // k-step's byte offset goes in the scalar offset)
  auto a_offsets = [&](int m0_, uint32_t (&va_)[SA]) {
#pragma unroll
    for (int i = 0; i < SA; ++i) {
      const int row = (wid * SA + i) * RPI + lr;
      const int ra = min(row, M - 1 - m0_);  // rows past M are computed on a copy and never stored
      va_[i] = (uint32_t)(ra * ldx + (lc ^ swz_a(row)) * EPC) * (uint32_t)ES;
    }
  };
  i32x4_t rA = buffer_rsrc(X + (int64_t)m0 * ldx), rB = buffer_rsrc(W + (int64_t)n0 * ldw);
  uint32_t va[SA], vb[SB];
  a_offsets(m0, va);
#pragma unroll
  for (int i = 0; i < SB; ++i) {
    const int row = (wid * SB + i) * RPI + lr;
    vb[i] = (uint32_t)(row * ldw + (lc ^ swz_b(row)) * EPC) * (uint32_t)ES;
  }
  // persistent: the next tile's origin, resources and A offsets (a copy of the
  // current tile's when there is none)
  int m0n = m0, n0n = n0;
  bool has_next = false;
  i32x4_t rAn = rA, rBn = rB;
  uint32_t van[SA];
#pragma unroll
  for (int i = 0; i < SA; ++i) van[i] = va[i];
  auto next_tile = [&]() {
    has_next = v + (int)gridDim.x < ntiles;
    if (has_next) {
      tile_origin(v + (int)gridDim.x, m0n, n0n);
      rAn = buffer_rsrc(X + (int64_t)m0n * ldx);
      rBn = buffer_rsrc(W + (int64_t)n0n * ldw);
      a_offsets(m0n, van);
    } else {
      m0n = m0;
      n0n = n0;
      rAn = rA;
      rBn = rB;
#pragma unroll
      for (int i = 0; i < SA; ++i) van[i] = va[i];
    }
  };
  if constexpr (PERSIST) next_tile();

  acc_t acc[TM][TN];
  auto zero_acc = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < NREG; ++r) acc[i][j][r] = 0.f;
  };
  zero_acc();

  const int nk = K / BK;
  // load instruction o (A rows for o < SA, then B rows) of k-step kt into
  // stage st. K-steps past the end reload the last one into a stage that is
  // never read again, so every step runs the same branch-free code; when
  // persistent, they are the next tile's first k-steps instead (the load stream
  // runs on across tiles, so the next tile's operands are in flight during this
  // tile's last steps and epilogue).
  auto issue_one = [&](int kt, auto stc, auto oc) {
    constexpr int st = decltype(stc)::value, o = decltype(oc)::value;
    if constexpr (PERSIST) {
      const bool nx = kt >= nk;  // uniform
      const uint32_t kb = (uint32_t)((nx ? (has_next ? kt - nk : nk - 1) : kt) * RB);
      if constexpr (o < SA)
        buffer_to_lds(nx ? rAn : rA, nx ? van[o] : va[o], kb, lds_addr(&sA[st][0]) + (wid * SA + o) * 1024);
      else
        buffer_to_lds(nx ? rBn : rB, vb[o - SA], kb, lds_addr(&sB[st][0]) + (wid * SB + o - SA) * 1024);
    } else {
      const uint32_t kb = (uint32_t)(min(kt, nk - 1) * RB);
      if constexpr (o < SA)
        buffer_to_lds(rA, va[o], kb, lds_addr(&sA[st][0]) + (wid * SA + o) * 1024);
      else
        buffer_to_lds(rB, vb[o - SA], kb, lds_addr(&sB[st][0]) + (wid * SB + o - SA) * 1024);
    }
  };
  u32x4_t fa[2][TM], fb[2][TN];
  // fragment read q (A fragment q for q < TM, then B) of sub-step kk of stage st
  auto read_one = [&](auto stc, int kk, auto qc, auto bufc) {
    constexpr int st = decltype(stc)::value, q = decltype(qc)::value, bf = decltype(bufc)::value;
    // lane l holds row l % T, chunk CPS kk + l / T
    const int ch = kk * CPS + lane / T;
    if constexpr (q < TM) {
      const int r = wm * WM + q * T + lane % T;
      fa[bf][q] = sA[st][r * CPR + (ch ^ swz_a(r))];
    } else {
      const int r = b_row(q - TM, lane % T);
      fb[bf][q - TM] = sB[st][r * CPR + (ch ^ swz_b(r))];
    }
  };
  // k-step kt: stage stc, next stage nstc, refilled stage rstc (k-step kt - 1's)
  auto step = [&](int kt, auto stc, auto nstc, auto rstc) {
    static_for<KK>([&](auto kkc) {
      constexpr int kk = decltype(kkc)::value;
      constexpr bool last = kk == KK - 1;
      constexpr int cur = kk & 1, nxt = (kk + 1) & 1;
      static_for<NU>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
        constexpr int m = u % NM, t = u / NM;
        if constexpr (last && u == UB) {
          wait_vmcnt_lds<(S - 2) * OPS>();
          lds_barrier();
        }
        if constexpr (F32)
          acc[m / TN][m % TN] = __builtin_amdgcn_mfma_f32_32x32x2f32(
              __uint_as_float(fa[cur][m / TN][t]), __uint_as_float(fb[cur][m % TN][t]), acc[m / TN][m % TN], 0, 0, 0);
        else
          acc[m / TN][m % TN] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8_t, fa[cur][m / TN]), __builtin_bit_cast(bf16x8_t, fb[cur][m % TN]),
              acc[m / TN][m % TN], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        static_for<NR>([&](auto qc) {
          constexpr int q = decltype(qc)::value;
          if constexpr (!last) {
            if constexpr (q * NU / NR == u) read_one(stc, kk + 1, qmap(qc), ic<nxt>{});
          } else if constexpr (u >= UB) {
            if constexpr (UB + q * (NU - UB) / NR == u) read_one(nstc, 0, qmap(qc), ic<0>{});
          }
        });
        constexpr int pos = kk * NU + u;
        static_for<OPS>([&](auto oc) {
          constexpr int o = decltype(oc)::value;
          if constexpr (o * LPOS / OPS == pos) issue_one(kt - 1 + S, rstc, oc);
        });
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };
  static_for<S - 1>([&](auto sc) { static_for<OPS>([&](auto oc) { issue_one(decltype(sc)::value, sc, oc); }); });
  wait_vmcnt_lds<(S - 2) * OPS>();
  lds_barrier();
  static_for<NR>([&](auto qc) { read_one(ic<0>{}, 0, qmap(qc), ic<0>{}); });
  auto group = [&](int kt) {  // S k-steps from a multiple of S
    static_for<S>([&](auto ic_) {
      constexpr int i = decltype(ic_)::value;
      step(kt + i, ic<i>{}, ic<(i + 1) % S>{}, ic<(i + S - 1) % S>{});
    });
  };

  // Bias and activation are applied per column; then each group of four
  // registers (four consecutive rows of one column) is transposed across the
  // four lanes of a quad, so that a lane holds four consecutive columns of one
  // row. fp32: register r of lane l is row 8 (r / 4) + 4 (l / 32) + r % 4, column
  // l % 32 of its 32 x 32 block. bf16: row 4 (l / 16) + r and row x = l % 16 of
  // the column block, which is column b_row(j, x): for bf16 outputs the two blocks
  // of a pair give a lane eight consecutive columns, stored at once (16 bytes);
  // for fp32 outputs two neighbouring blocks exchange halves, so that a store covers
  // 32 columns, a whole line, of eight rows (32768 x 512 x 1024 38.3 us, 32768 x
  // 1024 x 4096 237; with 16 columns of 16 rows a store 42.8 and 249, and 40.0 and
  // 234 on the 32x32x16 instruction, whose blocks are 32 columns wide).
  constexpr int NG = NREG / 4;                // groups of four registers per block
  constexpr int JS = F32 ? 1 : 2;             // column blocks stored at a time
  constexpr int NC = 4 * JS;                  // values a lane holds of them
  auto row_in = [&](int g) { return F32 ? 8 * g + 4 * (lane >> 5) + (lane & 3) : 4 * (lane >> 4) + (lane & 3); };
  // the lane's four columns of row block i, register group g of each of column blocks j .. j + JS - 1
  auto columns = [&](int i, int g, int j, const float (&bb)[JS], float (&q)[NC]) {
#pragma unroll
    for (int h = 0; h < JS; ++h) {
      float x[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = act_fn<ACT>(acc[i][j + h][4 * g + k] + bb[h]);
      quad_transpose4(x, lane);
#pragma unroll
      for (int k = 0; k < 4; ++k) q[4 * h + k] = x[k];
    }
  };
  auto first_col = [&](int j) { return b_row(j, lane & (T - 4)); };
  auto epilogue = [&]() {
  // with an output row map: the output offsets of this lane's rows, loaded
  // all at once before any is needed
  const bool mapped = OUT_F32 && om.rows != nullptr;  // uniform
  constexpr int NO = F32 ? NG : 2;                    // rows of a row block that a lane stores
  int64_t ro[TM][NO];
  // the lane's o-th row of a row block (fp32 outputs of a bf16 layer: after the exchange)
  auto out_row = [&](int o) { return F32 ? row_in(o) : 8 * o + 4 * ((lane >> 4) & 1) + (lane & 3); };
  if (mapped) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int o = 0; o < NO; ++o) {
        const int r = m0 + wm * WM + i * T + out_row(o);
        ro[i][o] = r < M ? om.rows[r].out : -1;
      }
  }
  // four fp32 columns from colq of the lane's o-th row of row block i. Streaming
  // (nontemporal) stores: the whole chip writes its tiles' outputs at about the
  // same time, and these drain faster than stores that allocate in L2
  auto store_f32 = [&](int i, int o, int colq, const float* q) {
    const int row = m0 + wm * WM + i * T + out_row(o);
    float* dst = nullptr;
    int n = 4;  // columns to store
    if (mapped) {
      if (ro[i][o] >= 0) dst = om.out + ro[i][o] + colq;
      n = min(4, om.d_out - colq);
    } else if (row < M) {
      dst = (float*)Y + (int64_t)row * ldy + colq;
    }
    if (!dst) return;
    if (n == 4 && ((uintptr_t)dst & 15) == 0) {
      const f32x4_t v = {q[0], q[1], q[2], q[3]};
      __builtin_nontemporal_store(v, (f32x4_t*)dst);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < n) dst[k] = q[k];
    }
  };
#pragma unroll
  for (int j = 0; j < TN; j += JS) {
    float bb[JS];
#pragma unroll
    for (int h = 0; h < JS; ++h) bb[h] = bias[n0 + b_row(j + h, lane % T)];
    const int colq = n0 + first_col(j);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        float q[NC];
        columns(i, g, j, bb, q);
        const int row = m0 + wm * WM + i * T + row_in(g);
        if constexpr (OUT_F32 && F32) {
          store_f32(i, g, colq, q);
        } else if constexpr (OUT_F32) {
          // the upper half of block j against the lower half of block j + 1: the
          // lanes then hold 32 columns of rows 0..7 in q[0..3], of rows 8..15 in q[4..7]
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(q[k]), __float_as_uint(q[4 + k]), false, false);
            q[k] = __uint_as_float(x[0]);
            q[4 + k] = __uint_as_float(x[1]);
          }
          const int c = colq + 16 * (lane >> 5);
          store_f32(i, 0, c, q);
          store_f32(i, 1, c, q + 4);
        } else if (row < M) {
          const u32x4_t o = {pack2_rne(q[0], q[1]), pack2_rne(q[2], q[3]), pack2_rne(q[4], q[5]), pack2_rne(q[6], q[7])};
          __builtin_nontemporal_store(o, (u32x4_t*)((bf16_t*)Y + (int64_t)row * ldy + colq));
        }
      }
  }
  };

  // The head instead of the store: the tile's outputs, rounded to bf16 exactly
  // as the store would round them, into LDS rows of HLD bytes (over the
  // operand stages, once every wave is done with them); then 16 lanes per row
  // sum w . y in the order of k_head (lane l: elements 8 l .. 8 l + 7 of every
  // 128, then a 16-lane butterfly), so the results equal the separate layer and
  // head bit for bit.
  auto head_epilogue = [&]() {
    if constexpr (HEAD >= 0) {
    constexpr int RPP = NT / 16;  // rows per pass of the head (16 lanes each)
    static_assert(!F32 && !OUT_F32 && BN == 256 && BM % RPP == 0, "bf16 layer of 256 outputs");
    constexpr int HLD = BN * 2 + 16;
    static_assert(BM * HLD <= S * BN * CPR * 16, "the output tile fits over the B stages");
    unsigned char* hb = (unsigned char*)&sB[0][0];
    // the output offsets of this thread's rows and its head weights, loaded
    // before the tile goes to LDS so that their latency overlaps it
    const int l = tid & 15;
    int64_t outs[BM / RPP];
#pragma unroll
    for (int p = 0; p < BM / RPP; ++p) {
      const int r = m0 + p * RPP + (tid >> 4);
      outs[p] = r < M ? ha.rows[r].out : -1;
    }
    const u32x4_t w0 = *(const u32x4_t*)(ha.w + l * 8), w1 = *(const u32x4_t*)(ha.w + 128 + l * 8);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TN; j += JS) {
      float bb[JS];
#pragma unroll
      for (int h = 0; h < JS; ++h) bb[h] = bias[n0 + b_row(j + h, lane % T)];
      const int colq = first_col(j);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          float q[NC];
          columns(i, g, j, bb, q);
          const int rl = wm * WM + i * T + row_in(g);
          const u32x4_t o = {pack2_rne(q[0], q[1]), pack2_rne(q[2], q[3]), pack2_rne(q[4], q[5]), pack2_rne(q[6], q[7])};
          *(u32x4_t*)(hb + rl * HLD + colq * 2) = o;
        }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < BM / RPP; ++p) {
      const int rl = p * RPP + (tid >> 4);
      float sum = 0.f;
      const int64_t o = outs[p];
      {
        if (o >= 0) {
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const u32x4_t hv = *(const u32x4_t*)(hb + rl * HLD + (c * 128 + l * 8) * 2), wv = c ? w1 : w0;
            sum += bf2f(hv.x & 0xffffu) * bf2f(wv.x & 0xffffu);
            sum += bf2f(hv.x >> 16) * bf2f(wv.x >> 16);
            sum += bf2f(hv.y & 0xffffu) * bf2f(wv.y & 0xffffu);
            sum += bf2f(hv.y >> 16) * bf2f(wv.y >> 16);
            sum += bf2f(hv.z & 0xffffu) * bf2f(wv.z & 0xffffu);
            sum += bf2f(hv.z >> 16) * bf2f(wv.z >> 16);
            sum += bf2f(hv.w & 0xffffu) * bf2f(wv.w & 0xffffu);
            sum += bf2f(hv.w >> 16) * bf2f(wv.w >> 16);
          }
        }
      }
      sum += __shfl_xor(sum, 1);
      sum += __shfl_xor(sum, 2);
      sum += __shfl_xor(sum, 4);
      sum += __shfl_xor(sum, 8);
      if (l == 0 && o >= 0) ha.out[o] = act_fn<HEAD>(sum + ha.b);
    }
    }
  };

  if constexpr (PERSIST) {
    // K a multiple of S k-steps (so every tile starts at stage 0) and at least
    // S k-steps (so the loads of a tile's last steps reach only the next tile)
    for (;;) {
      for (int kt = 0; kt < nk; kt += S) group(kt);
      epilogue();
      if (!has_next) break;
      v += gridDim.x;
      m0 = m0n;
      n0 = n0n;
      rA = rAn;
      rB = rBn;
#pragma unroll
      for (int i = 0; i < SA; ++i) va[i] = van[i];
      next_tile();
      zero_acc();
    }
    // no load into LDS may still be in flight when the wave ends
    wait_vmcnt_lds<0>();
  } else {
    int kt = 0;
    for (; kt + S <= nk; kt += S) group(kt);
    static_for<S - 1>([&](auto ic_) {
      constexpr int i = decltype(ic_)::value;
      if (kt + i < nk) step(kt + i, ic<i>{}, ic<(i + 1) % S>{}, ic<(i + S - 1) % S>{});
    });
    // no load into LDS may still be in flight when the wave ends
    wait_vmcnt_lds<0>();
    if constexpr (HEAD >= 0)
      head_epilogue();
    else
      epilogue();
  }
}

// The two operand types as separately named kernels (so that traces and
// counters tell them apart).
template <int BM, int BN, int WM, int WN, int NT, int RB, int S, int ACT, bool OUT_F32, bool PERSIST>
__global__ __launch_bounds__(NT) void k_gemm_bf16(const bf16_t* __restrict__ X, int ldx,
                                                  const bf16_t* __restrict__ W, int ldw,
                                                  const float* __restrict__ bias, void* __restrict__ Y, int ldy,
                                                  int M, int N, int K, int xcd_order, OutMap om) {
  gemm_mfma<bf16_t, BM, BN, WM, WN, NT, RB, S, ACT, OUT_F32, PERSIST>(X, ldx, W, ldw, bias, Y, ldy, M, N, K, xcd_order,
                                                                     nullptr, 0, HeadArgs{}, om);
}
// A bf16 layer of 256 outputs with a narrow head in its epilogue (HEAD: the
// head's activation); the layer's outputs never leave the workgroup.
template <int BM, int BN, int WM, int WN, int NT, int RB, int S, int ACT, int HEAD>
__global__ __launch_bounds__(NT) void k_gemm_head(const bf16_t* __restrict__ X, int ldx,
                                                  const bf16_t* __restrict__ W, int ldw,
                                                  const float* __restrict__ bias, int M, int K, HeadArgs ha) {
  gemm_mfma<bf16_t, BM, BN, WM, WN, NT, RB, S, ACT, false, false, HEAD>(X, ldx, W, ldw, bias, nullptr, BN, M,
                                                                       BN, K, 1, nullptr, 0, ha);
}
template <int BM, int BN, int WM, int WN, int NT, int RB, int S, int ACT>
__global__ __launch_bounds__(NT) void k_gemm_f32(const float* __restrict__ X, int ldx, const float* __restrict__ W,
                                                 int ldw, const float* __restrict__ bias, void* __restrict__ Y,
                                                 int ldy, int M, int N, int K, int xcd_order,
                                                 const rb_k_row* __restrict__ skip_rows, int skip_T, OutMap om) {
  gemm_mfma<float, BM, BN, WM, WN, NT, RB, S, ACT, true, false>(X, ldx, W, ldw, bias, Y, ldy, M, N, K, xcd_order,
                                                               skip_rows, skip_T, HeadArgs{}, om);
}

// PERSIST: a grid of at most `cap` workgroups (a multiple of 8), each taking
// every cap-th tile
template <typename TI, int BM, int BN, int WM, int WN, int NT, int RB, int S, bool PERSIST = false>
void launch_gemm(hipStream_t s, const TI* x, int ldx, const TI* w, int ldw, const float* b, void* Y, int ldy,
                 int M, int N, int K, int act, bool out_f32, int xcd, const rb_k_row* skip_rows, int skip_T,
                 unsigned cap = 0, OutMap om = OutMap{}) {
  const unsigned tiles = (unsigned)(((M + BM - 1) / BM) * (N / BN));
  const unsigned g = PERSIST ? std::min(tiles, cap) : tiles;
  if constexpr (sizeof(TI) == 4) {
#define RB_G(A)                                                                                                     \
  hipLaunchKernelGGL((k_gemm_f32<BM, BN, WM, WN, NT, RB, S, A>), dim3(g), dim3(NT), 0, s, x, ldx, w, ldw, b, \
                     Y, ldy, M, N, K, xcd, skip_rows, skip_T, om)
    if (act == RB_ACT_RELU) RB_G(RB_ACT_RELU);
    else if (act == RB_ACT_SIGMOID) RB_G(RB_ACT_SIGMOID);
    else RB_G(RB_ACT_NONE);
#undef RB_G
  } else {
#define RB_G(A, F)                                                                                             \
  hipLaunchKernelGGL((k_gemm_bf16<BM, BN, WM, WN, NT, RB, S, A, F, PERSIST>), dim3(g), dim3(NT), 0, s, x, ldx, w, \
                     ldw, b, Y, ldy, M, N, K, xcd, om)
    if (out_f32) {
      if (act == RB_ACT_RELU) RB_G(RB_ACT_RELU, true);
      else if (act == RB_ACT_SIGMOID) RB_G(RB_ACT_SIGMOID, true);
      else RB_G(RB_ACT_NONE, true);
    } else {
      if (act == RB_ACT_RELU) RB_G(RB_ACT_RELU, false);
      else if (act == RB_ACT_SIGMOID) RB_G(RB_ACT_SIGMOID, false);
      else RB_G(RB_ACT_NONE, false);
    }
#undef RB_G
  }
}

}  // namespace

extern "C" {

namespace {
rb_status gemm_bf16_impl(void* stream, const void* X, int32_t ldx, const void* W, int32_t ldw, const float* b,
                         void* Y, int32_t ldy, int32_t M, int32_t N, int32_t K, int32_t act, int32_t out_f32,
                         OutMap om) {
  if (M < 0 || N <= 0 || K <= 0 || (N % 128) || (K % G16_KALIGN) || ldx < K || ldw < K) return RB_EINVAL;
  if ((ldx & 7) || (ldw & 7) || !X || !W || !b) return RB_EINVAL;
  // operand byte offsets within a 256-row tile are 32-bit
  if ((int64_t)ldx * 512 >= ((int64_t)1 << 31) || (int64_t)ldw * 512 >= ((int64_t)1 << 31)) return RB_EINVAL;
  if (act != RB_ACT_NONE && act != RB_ACT_RELU && act != RB_ACT_SIGMOID) return RB_EINVAL;
  if (M == 0) return RB_OK;
  hipStream_t s = (hipStream_t)stream;
  const bf16_t* x = (const bf16_t*)X;
  const bf16_t* w = (const bf16_t*)W;
  // Tile shape, k-step, stage count and tile order only change speed: every
  // choice accumulates each output in the same k order with the same
  // instruction (identical bits). The largest tile that still gives every CU a
  // tile: 256 x 256 (8 waves of 64 x 128, k-step 64, 2 stages, 128 KB LDS, every
  // row's k-step a whole 128-byte line; 4 waves of 128 x 128 need every register
  // and measured 1.3x slower), else 256 x 128 (8 waves of 64 x 64, k-step 64, 3
  // stages, 144 KB), else
  // 128 x 128 (8 waves of 64 x 32, k-step 64, 4 stages, 128 KB) or smaller ones
  // for launches of few rows. XCD-contiguous
  // tile order when all of W fits in one XCD's L2 (each XCD then keeps its A
  // row-blocks and W in its own L2); plain order otherwise (contiguous ranges
  // would stream all of W through every XCD).
  //
  // With more 256 x 128 tiles than compute units, the grid is persistent (one
  // workgroup per CU, each taking every CU-count-th tile) when K is a multiple of the
  // stage count in k-steps: the operand loads then run on across tile
  // boundaries, so a tile's first k-steps load during the previous tile's last
  // steps and epilogue.
  const int64_t rows256 = (M + 255) / 256;
  const bool xcd = (int64_t)N * K * 2 <= (4 << 20);
  const unsigned cus = device_cus() & ~7u;
#define RB_PICK(BM, BN, WM, WN, NT, BK, S, P)                                                                      \
  launch_gemm<bf16_t, BM, BN, WM, WN, NT, BK * 2, S, P>(s, x, ldx, w, ldw, b, Y, ldy, M, N, K, act, out_f32 != 0, xcd, \
                                                        nullptr, 0, cus, om)
  auto persist = [&](int bm, int bn, int bk, int st) {
    const int64_t tiles = ((M + bm - 1) / bm) * (int64_t)(N / bn);
    const int nk = K / bk;
    return cus >= 8 && tiles > (int64_t)cus && nk >= st && nk % st == 0;
  };
  if (N % 256 == 0 && rows256 * (N / 256) >= 256) {
    RB_PICK(256, 256, 64, 128, 512, 64, 2, false);
  } else if (rows256 * (N / 128) >= 256) {
    if (persist(256, 128, 64, 3))
      RB_PICK(256, 128, 64, 64, 512, 64, 3, true);
    else
      RB_PICK(256, 128, 64, 64, 512, 64, 3, false);
  } else {
    // fewer tiles than that. A wave issues its loads, LDS reads and MFMAs one
    // after another, and a compute unit's loads enter at 64 bytes a clock, so a
    // launch of few rows takes as long as one tile's k-loop: the smallest tiles
    // that still leave one to a compute unit, and 128 x 64 once 64 x 64 would be
    // two. Back to back, us, with W from HBM (and on one W, from the caches):
    //                     32 x 32      64 x 32      64 x 64      128 x 64     128 x 128
    //   64 x 1024 x 1728   6.0 (6.2)    6.3 (6.4)    7.5 (6.9)    8.9 (8.9)  10.7 (10.6)
    //   512 x 1024 x 1728  7.8 (7.0)    7.3 (6.8)    8.1 (7.7)    9.9 (9.0)  12.6 (11.1)
    //   64 x 8192 x 8192                40 (33)      45 (29)      47 (33)      61 (39)
    //   128 x 8192 x 8192  81 (68)      67 (63)      45 (36)      56 (41)      75 (44)
    //   256 x 8192 x 8192                            70 (55)      57 (43)      76 (44)
    //   512 x 3072 x 3008               27 (24)      20 (19)      21 (16)      30 (20)
    //   1024 x 2048 x 2048                           16.2 (14.8)  12.5 (12.5)  14.8 (15.1)
    //   2816 x 512 x 1024                                 (7.4)        (7.1)
    // (64 x 64 tiles with two waves of 64 x 32 instead of four of 32 x 32: 15.1
    // (14.2) for 1024 x 2048 x 2048, 63 (46) for 256 x 8192 x 8192)
    const int64_t rows64 = (M + 63) / 64, rows32 = (M + 31) / 32;
    if (rows32 * (N / 32) <= (int64_t)cus)
      RB_PICK(32, 32, 32, 32, 64, 64, 6, false);
    else if (rows64 * (N / 32) <= (int64_t)cus)
      RB_PICK(64, 32, 32, 32, 128, 64, 8, false);
    else if (rows64 * (N / 64) <= (int64_t)cus)
      RB_PICK(64, 64, 32, 32, 256, 64, 4, false);
    else if (rows64 * (N / 64) <= 2 * (int64_t)cus)
      RB_PICK(128, 64, 64, 32, 256, 64, 4, false);
    else
      RB_PICK(128, 128, 64, 32, 512, 64, 4, false);
  }
#undef RB_PICK
  return launch_status();
}
}  // namespace

rb_status rb_k_gemm_bf16(void* stream, const void* X, int32_t ldx, const void* W, int32_t ldw, const float* b,
                         void* Y, int32_t ldy, int32_t M, int32_t N, int32_t K, int32_t act, int32_t out_f32) {
  if (ldy < N || (ldy & 7) || ((uintptr_t)Y & 15) || !Y) return RB_EINVAL;
  return gemm_bf16_impl(stream, X, ldx, W, ldw, b, Y, ldy, M, N, K, act, out_f32, OutMap{});
}

rb_status rb_k_gemm_bf16_rows(void* stream, const void* X, int32_t ldx, const void* W, int32_t ldw, const float* b,
                              int32_t M, int32_t N, int32_t K, int32_t act, const rb_k_row* rows, int32_t d_out,
                              float* out) {
  if (!rows || !out || d_out < 1 || d_out > N) return RB_EINVAL;
  return gemm_bf16_impl(stream, X, ldx, W, ldw, b, nullptr, N, M, N, K, act, 1, OutMap{rows, out, d_out});
}

namespace {
rb_status gemm_f32_impl(void* stream, const float* X, int32_t ldx, const float* W, int32_t ldw, const float* b,
                        float* Y, int32_t ldy, int32_t M, int32_t N, int32_t K, int32_t act,
                        const rb_k_row* skip_rows, int32_t skip_T, OutMap om) {
  if (M < 0 || N <= 0 || K <= 0 || (N % 64) || (K % G32_KALIGN) || ldx < K || ldw < K) return RB_EINVAL;
  if ((ldx & 3) || (ldw & 3) || !X || !W || !b) return RB_EINVAL;
  if (((uintptr_t)X & 15) || ((uintptr_t)W & 15)) return RB_EINVAL;
  // operand byte offsets within a 64-row tile are 32-bit
  if ((int64_t)ldx * 4 * G32_BM >= ((int64_t)1 << 31) || (int64_t)ldw * 4 * 64 >= ((int64_t)1 << 31)) return RB_EINVAL;
  if (act != RB_ACT_NONE && act != RB_ACT_RELU && act != RB_ACT_SIGMOID) return RB_EINVAL;
  if (skip_rows && (skip_T <= 0 || skip_T % G32_BM)) return RB_EINVAL;
  if (M == 0) return RB_OK;
  hipStream_t s = (hipStream_t)stream;
  // 64 x 64 tiles (64 rows: the padding-token skip granularity), 4 waves of
  // 32 x 32, k-step 16, 3 stages (24 KB LDS, six workgroups per CU). Small
  // wave tiles keep the work per wave small, so the CUs stay evenly loaded when
  // padding-token blocks leave holes in the grid (64 x 64 wave tiles measured
  // up to 1.5x slower there). XCD-contiguous tile order when W fits in one
  // XCD's L2 (each XCD then reads its X rows once; plain order measured 1.5x
  // slower on sequence groups).
  const bool xcd = (int64_t)N * K * 4 <= (4 << 20);
  launch_gemm<float, G32_BM, 64, 32, 32, 256, 64, 3>(s, X, ldx, W, ldw, b, Y, ldy, M, N, K, act, true, xcd, skip_rows,
                                                     skip_T, 0, om);
  return launch_status();
}
}  // namespace

rb_status rb_k_gemm_f32(void* stream, const float* X, int32_t ldx, const float* W, int32_t ldw, const float* b,
                        float* Y, int32_t ldy, int32_t M, int32_t N, int32_t K, int32_t act,
                        const rb_k_row* skip_rows, int32_t skip_T) {
  if (ldy < N || (ldy & 3) || ((uintptr_t)Y & 15) || !Y) return RB_EINVAL;
  return gemm_f32_impl(stream, X, ldx, W, ldw, b, Y, ldy, M, N, K, act, skip_rows, skip_T, OutMap{});
}

rb_status rb_k_gemm_f32_rows(void* stream, const float* X, int32_t ldx, const float* W, int32_t ldw, const float* b,
                             int32_t M, int32_t N, int32_t K, int32_t act, const rb_k_row* rows, int32_t d_out,
                             float* out) {
  if (!rows || !out || d_out < 1 || d_out > N) return RB_EINVAL;
  return gemm_f32_impl(stream, X, ldx, W, ldw, b, nullptr, N, M, N, K, act, nullptr, 0, OutMap{rows, out, d_out});
}

rb_status rb_k_gemm_head(void* stream, const void* X, int32_t ldx, const void* W, int32_t ldw, const float* b,
                         int32_t M, int32_t K, int32_t act, const rb_k_row* rows, const void* w_head, float b_head,
                         int32_t head_act, float* out) {
  if (M < 0 || K <= 0 || (K % G16_KALIGN) || ldx < K || ldw < K || (ldx & 7) || (ldw & 7)) return RB_EINVAL;
  if (!X || !W || !b || !rows || !w_head || !out || ((uintptr_t)w_head & 15)) return RB_EINVAL;
  if ((int64_t)ldx * 512 >= ((int64_t)1 << 31) || (int64_t)ldw * 512 >= ((int64_t)1 << 31)) return RB_EINVAL;
  if (act != RB_ACT_NONE && act != RB_ACT_RELU && act != RB_ACT_SIGMOID) return RB_EINVAL;
  if (head_act != RB_ACT_NONE && head_act != RB_ACT_SIGMOID) return RB_EINVAL;
  if (M == 0) return RB_OK;
  // 128 x 256 tiles (every row's 256 outputs in one workgroup), 8 waves of
  // 64 x 64 (two per SIMD: 4 waves of 64 x 128 measured 16% slower), k-step
  // 64, 3 stages; XCD-contiguous order (W is 256 x K bf16). With fewer such
  // tiles than half the compute units (a launch of a few batches, bound by
  // its k-loop's latency), 64 x 256 tiles of 8 waves of 64 x 32.
  const bool small = (int64_t)(M + 127) / 128 < std::max<int64_t>(device_cus() / 2, 1);
  const unsigned g = (unsigned)(small ? (M + 63) / 64 : (M + 127) / 128);
  const HeadArgs ha{rows, (const bf16_t*)w_head, b_head, out};
  hipStream_t s = (hipStream_t)stream;
#define RB_GH(A, H)                                                                                                    \
  do {                                                                                                                 \
    if (small)                                                                                                         \
      hipLaunchKernelGGL((k_gemm_head<64, 256, 64, 32, 512, 128, 3, A, H>), dim3(g), dim3(512), 0, s,             \
                         (const bf16_t*)X, ldx, (const bf16_t*)W, ldw, b, M, K, ha);                                   \
    else                                                                                                               \
      hipLaunchKernelGGL((k_gemm_head<128, 256, 64, 64, 512, 128, 3, A, H>), dim3(g), dim3(512), 0, s,            \
                         (const bf16_t*)X, ldx, (const bf16_t*)W, ldw, b, M, K, ha);                                   \
  } while (0)
  if (head_act == RB_ACT_SIGMOID) {
    if (act == RB_ACT_RELU) RB_GH(RB_ACT_RELU, RB_ACT_SIGMOID);
    else if (act == RB_ACT_SIGMOID) RB_GH(RB_ACT_SIGMOID, RB_ACT_SIGMOID);
    else RB_GH(RB_ACT_NONE, RB_ACT_SIGMOID);
  } else {
    if (act == RB_ACT_RELU) RB_GH(RB_ACT_RELU, RB_ACT_NONE);
    else if (act == RB_ACT_SIGMOID) RB_GH(RB_ACT_SIGMOID, RB_ACT_NONE);
    else RB_GH(RB_ACT_NONE, RB_ACT_NONE);
  }
#undef RB_GH
  return launch_status();
}

}  // extern "C"
