// Device kernels of the batched inference path, written for gfx950 (CDNA4,
// wave64, MFMA, 160 KB LDS per CU).
//
// A launch group is a set of dispatched batches of one queue. Its rows live in
// one row space: batch b owns rows [row_base_b, row_base_b + P_b), the first
// s_b of them real, the rest padding (the batch axis padded to an allowed
// size). The kernels, in the order a group runs them:
//
//   route     per-batch exclusive prefix scans: which request row (or padding)
//             every row is, where its input and output live (the paper's
//             concatenation of input tensors, section 2.2.1, as an index map),
//             and where each of its embedding bags ends
//   assemble  gather request rows into the padded batch tensor (optional
//             fp32 -> bf16 cast), or
//   embbag    sum-pool each row's embedding bags (ranking models)
//   gemm      dense layers with fused bias + activation (bf16 or fp32 MFMA);
//             the last layer of a chain without a head writes its real rows
//             straight into the requests' outputs through the row map (the
//             split fused in)
//   gemm_head the last hidden layer of 256 outputs and a narrow head in one
//             kernel, or
//   head /    narrow last layer or masked mean-pool + softmax head, writing
//   seqpool   straight to each request's output rows
//   split     copy real rows to their requests' outputs (padding dropped;
//             the unfused form, kept for the C ABI)
//
// Every row is computed the same way whatever batch it sits in (one tile
// shape and k order per layer, no row-count-dependent split of the sum), so a
// request's result does not depend on how its batch was composed.
#include <mutex>

#include "device.h"
#include "launch.h"

namespace {

// ---------------------------------------------------------------- route

constexpr int ROUTE_MAX_ROWS = 4096;  // rows (sequence slots) per batch
constexpr int ROUTE_NT = 512;         // threads per batch

// Block-wide exclusive scan of one value per thread (ROUTE_NT threads);
// returns the exclusive prefix and writes the block total to *total.
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T* s_w, T* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  T incl = v;
  for (int o = 1; o < 64; o <<= 1) {
    const T u = __shfl_up(incl, o);
    if (lane >= o) incl += u;
  }
  if (lane == 63) s_w[wid] = incl;
  __syncthreads();
  T off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < ROUTE_NT / 64; ++w) {
    if (w < wid) off += s_w[w];
    tot += s_w[w];
  }
  *total = tot;
  __syncthreads();
  return off + incl - v;
}

// Whether a batch's rows and requests lie inside the row map and the request
// table (its rows are otherwise not written).
__device__ __forceinline__ bool batch_in_range(const rb_k_batch& b, int max_rows, int n_rows_total, int n_reqs) {
  return b.padded <= max_rows && b.n_req <= b.padded && b.real <= b.padded && b.padded >= 0 && b.n_req >= 0 &&
         b.row_base >= 0 && (int64_t)b.row_base + b.padded <= n_rows_total && b.req_begin >= 0 &&
         (int64_t)b.req_begin + b.n_req <= n_reqs;
}

// One workgroup per batch, all steps parallel over requests or rows. A launch
// waits for one chain of dependent loads (the batch, its requests' row counts,
// a row's request, its lengths), so:
//  1. exclusive scan of the requests' row counts -> each request's first row
//     (the concatenation offsets), and a row -> request map in LDS;
//  2. per real row, its request's descriptor, kept in registers for the first
//     ROUTE_NT rows, and its id count (ranking: sum of its bag lengths) or token
//     count (seqpool: its sequence length). The lengths are loaded 16 bytes at a
//     time, 8 loads in flight (one length per load touched 64 lines 26 times
//     a wave). When `ends` is given, ends[f n_rows_total + row] is the end of the
//     row's bag f among its ids, so that the embedding kernel finds a bag with
//     two loads;
//  3. exclusive scan of those counts over the batch's rows; a row's first id
//     (token) is its request's base plus the scan difference to the request's
//     first row; each request is checked against its payload extent;
//  4. the row map entries, then padding rows. A sequence's entry also names
//     the row of its first token when the group's real tokens are packed
//     (its request's first packed row, set by the host, plus the scan).
// MAXR: the largest batch (512 rows take 7 KB of LDS, so that the workgroups
// find a place beside another stream's GEMM; 4096 take 54). Beside other
// streams' kernels 64 batches of 512 rows take 11.1 us at least, against 12.4
// without the ends; with a GEMM's worth of LDS for coalesced staging of the
// lengths it was 16.8.
// fill: the rows that no batch in range covers are set to padding too: each
// batch's workgroup sets those from its end to the next batch's start (the
// first one also those before it; without any, the first workgroup all). Every
// workgroup reads every batch for it, so the launch does so for up to ROUTE_NT
// batches, a descriptor a thread; more take a launch of their own first
// (k_fill_rows). One-row batches of a 64-128-16 MLP, us for the whole group by
// the routing launch and with a launch of its own: 1024 batches 25.6 and 18.8,
// 8192 409 and 48, 65536 22770 and 341; up to 512 a launch costs more than it
// reads (an idle server's ranking request: 2.5 of 36 us).
template <int MAXR>
__global__ __launch_bounds__(ROUTE_NT) void k_route(int kind, const rb_k_batch* __restrict__ batches, int n_batches,
                                                    const rb_k_req* __restrict__ reqs, int n_reqs,
                                                    const int32_t* __restrict__ lens, int64_t lens_len, int d_in,
                                                    int d_out, int n_tables, rb_k_row* __restrict__ rows,
                                                    int n_rows_total, int64_t out_len, int32_t* __restrict__ ends,
                                                    int fill, int* __restrict__ err) {
  const rb_k_batch b = batches[blockIdx.x];
  const int tid = threadIdx.x;
  __shared__ uint16_t s_first[MAXR + 1];   // first row of request i (batch-relative)
  __shared__ uint16_t s_req[MAXR];         // request of row p
  __shared__ int64_t s_ex[MAXR + 1];       // exclusive scan of per-row id/token counts
  __shared__ unsigned char s_bad[MAXR];
  __shared__ int64_t s_w[ROUTE_NT / 64];
  __shared__ int s_w32[ROUTE_NT / 64];
  __shared__ int s_desc_bad, s_next, s_prev;
  const rb_k_row none = {-1, 0, -1, -1};
  const bool in_range = batch_in_range(b, MAXR, n_rows_total, n_reqs);  // uniform
  if (tid == 0) {
    s_desc_bad = 0;
    s_next = n_rows_total;
    s_prev = 0;
    if (!in_range) *err = 1;
  }
  __syncthreads();
  if (fill) {
    // s_next: where the rows that another batch covers or fills start after
    // this one's end (of empty batches at one row the last in the list fills);
    // s_prev: whether any batch in range comes before it
    const int end = in_range ? b.row_base + b.padded : 0;
    for (int i = tid; i < n_batches; i += ROUTE_NT) {
      const rb_k_batch o = batches[i];
      if (i == (int)blockIdx.x || !batch_in_range(o, MAXR, n_rows_total, n_reqs)) continue;
      if (o.row_base > end || (o.row_base == end && (o.padded > 0 || i > (int)blockIdx.x)))
        atomicMin(&s_next, o.row_base);
      else if (o.row_base < end && o.row_base + o.padded > end)
        atomicMin(&s_next, end);
      if (o.row_base < b.row_base || (o.row_base == b.row_base && i < (int)blockIdx.x) || !in_range) s_prev = 1;
    }
    __syncthreads();
    if (in_range) {
      for (int r = end + tid; r < s_next; r += ROUTE_NT) rows[r] = none;
      if (!s_prev)
        for (int r = tid; r < b.row_base; r += ROUTE_NT) rows[r] = none;
    } else if (!s_prev && blockIdx.x == 0) {
      for (int r = tid; r < n_rows_total; r += ROUTE_NT) rows[r] = none;
    }
  }
  if (!in_range) return;
  // 1. request offsets
  int s = 0;
  for (int base = 0; base < b.n_req; base += ROUTE_NT) {
    const int i = base + tid;
    int n = i < b.n_req ? reqs[b.req_begin + i].n_rows : 0;
    if (i < b.n_req && (n < 1 || n > MAXR)) {  // every request has >= 1 row
      s_desc_bad = 1;
      n = 0;
    }
    int tot;
    const int ex = block_exclusive_scan(n, s_w32, &tot);
    if (i < b.n_req && s + ex <= MAXR) {
      s_first[i] = (uint16_t)(s + ex);
      s_bad[i] = 0;
    }
    s += tot;
  }
  __syncthreads();
  if (s > b.padded || s_desc_bad) {  // uniform
    if (tid == 0) *err = 1;
    if (fill)
      for (int p = tid; p < b.padded; p += ROUTE_NT) rows[b.row_base + p] = none;
    return;
  }
  if (tid == 0) s_first[b.n_req] = (uint16_t)s;
  __syncthreads();
  for (int i = tid; i < b.n_req; i += ROUTE_NT)
    for (int p = s_first[i]; p < s_first[i + 1]; ++p) s_req[p] = (uint16_t)i;
  __syncthreads();
  // 2 + 3. per-row counts and their scan
  rb_k_req rq0 = {};  // the descriptor of row tid's request
  int64_t carry = 0;
  for (int base = 0; base < s; base += ROUTE_NT) {
    const int p = base + tid;
    int64_t c = 0;
    if (p < s) {
      const int i = s_req[p];
      const rb_k_req rq = reqs[b.req_begin + i];
      if (base == 0) rq0 = rq;
      const int e = p - s_first[i];
      // a request whose output rows would lie outside the output, or whose bag
      // or sequence lengths outside the lens arena, is rejected
      const int64_t nl = kind == RB_MODEL_RANKING ? (int64_t)rq.n_rows * n_tables
                                                  : (kind == RB_MODEL_SEQPOOL ? rq.n_rows : 0);
      const bool in_arena = e < rq.n_rows && rq.out_off >= 0 && rq.out_off + (int64_t)rq.n_rows * d_out <= out_len &&
                            (nl == 0 || (rq.lens_off >= 0 && rq.lens_off + nl <= lens_len));
      if (!in_arena) {
        s_bad[i] = 1;
      } else if (kind == RB_MODEL_RANKING) {
        typedef int i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
        const int32_t* l = lens + rq.lens_off + (int64_t)e * n_tables;
        int32_t* en = ends ? ends + b.row_base + p : nullptr;
        // 32-bit sums while every length is under 2^25 (64 tables then stay under
        // 2^31): 64-bit ones with a test for negative lengths took 5.6 us for 8
        // rows of 26 bags (5.5 this way), 7.8 for 512 batches of 16 rows of 64 (7.5)
        uint32_t any = 0, sum = 0;  // the lengths' bits, their sum
        for (int f0 = 0; f0 < n_tables; f0 += 32) {
          uint32_t v[32];
#pragma unroll
          for (int u = 0; u < 32; u += 4) {
            const int f = f0 + u;
            if (f + 4 <= n_tables) {
              const i32x4_any q = *(const i32x4_any*)(l + f);
              v[u] = q[0]; v[u + 1] = q[1]; v[u + 2] = q[2]; v[u + 3] = q[3];
            } else {
#pragma unroll
              for (int k = 0; k < 4; ++k) v[u + k] = f + k < n_tables ? l[f + k] : 0;
            }
          }
#pragma unroll
          for (int u = 0; u < 32; ++u) {
            any |= v[u];
            sum += v[u];
            if (en && f0 + u < n_tables) en[(int64_t)(f0 + u) * n_rows_total] = (int32_t)sum;
          }
        }
        c = sum;
        if (any >> 25) {
          c = 0;
          for (int f = 0; f < n_tables; ++f) {
            if (l[f] < 0) s_bad[i] = 1;
            c += l[f];
            if (en) en[(int64_t)f * n_rows_total] = (int32_t)c;
          }
          if (c > INT32_MAX) s_bad[i] = 1;
        }
      } else if (kind == RB_MODEL_SEQPOOL) {
        const int v = lens[rq.lens_off + e];
        if (v < 1 || v > b.seq_T) s_bad[i] = 1;
        c = v;
      }
    }
    if (kind == RB_MODEL_MLP) continue;
    int64_t tot;
    const int64_t ex = block_exclusive_scan(c, s_w, &tot);
    if (p < s) s_ex[p] = carry + ex;
    carry += tot;
  }
  if (tid == 0) s_ex[s] = carry;
  __syncthreads();
  // 4. row entries
  for (int p = tid; p < b.padded; p += ROUTE_NT) {
    rb_k_row rw = none;
    if (p < s) {
      const int i = s_req[p], p0 = s_first[i], p1 = s_first[i + 1];
      const rb_k_req rq = p == tid ? rq0 : reqs[b.req_begin + i];
      const int e = p - p0;
      const int64_t cnt = kind == RB_MODEL_MLP ? 0 : s_ex[p1] - s_ex[p0];
      const int64_t within = kind == RB_MODEL_MLP ? 0 : s_ex[p] - s_ex[p0];
      bool ok = !s_bad[i];
      ok = ok && (kind == RB_MODEL_SEQPOOL ? cnt : (int64_t)(p1 - p0)) * d_in == rq.dense_end - rq.dense_off;
      if (kind == RB_MODEL_RANKING) ok = ok && cnt == rq.ids_end - rq.ids_off;
      if (!ok) *err = 1;
      if (kind == RB_MODEL_SEQPOOL) {
        rw.src = ok ? rq.dense_off + within * d_in : -1;
        rw.aux = ok ? s_ex[p + 1] - s_ex[p] : 0;
        rw.lens = ok ? rq.tok_off + within : -1;  // first row among the group's packed tokens
      } else {
        rw.src = ok ? rq.dense_off + (int64_t)e * d_in : -1;
        rw.aux = rq.ids_off + within;
        rw.lens = (kind == RB_MODEL_RANKING && ok) ? rq.lens_off + (int64_t)e * n_tables : -1;
      }
      rw.out = ok ? rq.out_off + (int64_t)e * d_out : -1;  // a rejected request's rows are not returned
    }
    rows[b.row_base + p] = rw;
  }
}

// Every row of a group's row space as padding.
__global__ __launch_bounds__(256) void k_fill_rows(rb_k_row* __restrict__ rows, int n) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r < n) rows[r] = rb_k_row{-1, 0, -1, -1};
}

// ---------------------------------------------------------------- assemble

// One thread per 8 output elements of a row: coalesced 16-byte stores of the
// padded batch tensor. Padding rows (and padding tokens) get `pad` in their
// d_in input columns; columns past d_in are always zero so that they add
// nothing in the next contraction.
// Real tokens only (sequence slots): workgroup (e, j) copies tokens
// [16 j, 16 j + 16) of slot e that lie below its length L (8 columns per thread
// and chunk, two chunks in flight, columns past d_in zeroed); blocks past L,
// rows t >= L and padding slots are not written (8..64-token blocks and 1..4
// chunks in flight measured no faster). Token t goes to row e T + t of X, or,
// with PACKED, to row rows[e].lens + t of the group's packed tokens (x_rows
// rows). lg_c = log2(ldx / 8) when that is a power of two, else -1.
constexpr int SEQ_TOK = 16, SEQ_U = 2;
template <bool PACKED>
__global__ __launch_bounds__(256) void k_assemble_seq(const rb_k_row* __restrict__ rows, int T,
                                                      const float* __restrict__ dense, int64_t dense_len, int d_in,
                                                      float* __restrict__ X, int ldx, int64_t x_rows,
                                                      int* __restrict__ err, int lg_c) {
  const rb_k_row rw = rows[blockIdx.x];
  const int t0 = blockIdx.y * SEQ_TOK;
  if (rw.src < 0 || t0 >= rw.aux) return;
  const int64_t L = rw.aux;
  if (L > T || rw.src + L * d_in > dense_len || (PACKED && (rw.lens < 0 || rw.lens + L > x_rows))) {
    if (threadIdx.x == 0) *err = 1;
    return;
  }
  const int cpr = ldx >> 3;
  const int n_tok = (int)min((int64_t)SEQ_TOK, L - t0);
  const int total = n_tok * cpr;
  const float* src = dense + rw.src + (int64_t)t0 * d_in;
  float* xb = X + ((PACKED ? rw.lens : (int64_t)blockIdx.x * T) + t0) * ldx;
  const bool vec = (d_in & 3) == 0 && (rw.src & 3) == 0;
  // SEQ_U chunks per thread and step: all loads issued before the stores
  for (int base = threadIdx.x; base < total; base += 256 * SEQ_U) {
    float v[SEQ_U][8];
#pragma unroll
    for (int u = 0; u < SEQ_U; ++u) {
      const int i = base + 256 * u;
      if (i >= total) break;
      const int t = lg_c >= 0 ? i >> lg_c : i / cpr;
      const int c0 = (i - t * cpr) * 8;
      const float* sr = src + (int64_t)t * d_in;
      if (vec) {
#pragma unroll
        for (int h = 0; h < 8; h += 4) {
          if (c0 + h < d_in) {
            const float4 a = *(const float4*)(sr + c0 + h);
            v[u][h] = a.x; v[u][h + 1] = a.y; v[u][h + 2] = a.z; v[u][h + 3] = a.w;
          } else {
            v[u][h] = v[u][h + 1] = v[u][h + 2] = v[u][h + 3] = 0.f;
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[u][j] = (c0 + j < d_in) ? sr[c0 + j] : 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < SEQ_U; ++u) {
      const int i = base + 256 * u;
      if (i >= total) break;
      const int t = lg_c >= 0 ? i >> lg_c : i / cpr;
      const int c0 = (i - t * cpr) * 8;
      float* y = xb + (int64_t)t * ldx + c0;
      *(float4*)y = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
      *(float4*)(y + 4) = make_float4(v[u][4], v[u][5], v[u][6], v[u][7]);
    }
  }
}

// One thread per 8 consecutive columns of one row (one 16-byte bf16 store or
// two fp32 ones; 4 or 16 columns measured slower). POW2: ldx / 8 and seq_T
// (when non-zero) are powers of two and the thread count fits 31 bits, so the
// row, chunk and slot indices come from shifts (lg_c = log2(ldx / 8), lg_t =
// log2(seq_T)); otherwise 64-bit division.
template <bool BF16, bool POW2>
__global__ __launch_bounds__(256) void k_assemble(const rb_k_row* __restrict__ rows, int n_rows_total,
                                                  int seq_T, const float* __restrict__ dense,
                                                  int64_t dense_len, int d_in, void* __restrict__ X,
                                                  int ldx, float pad, int* __restrict__ err, int lg_c, int lg_t) {
  constexpr int E = 8;
  const int chunks = ldx / E;
  int64_t r;
  int c0;
  if (POW2) {
    const uint32_t gid = blockIdx.x * 256u + threadIdx.x;
    r = (int64_t)(gid >> lg_c);
    c0 = (int)(gid & (uint32_t)(chunks - 1)) * E;
  } else {
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    r = gid / chunks;
    c0 = (int)(gid - r * chunks) * E;
  }
  if (r >= n_rows_total) return;
  int64_t src;
  if (seq_T > 0) {
    const int64_t slot = POW2 ? (int64_t)((uint32_t)r >> lg_t) : r / seq_T;
    const int t = (int)(r - slot * seq_T);
    const rb_k_row rw = rows[slot];
    src = (rw.src >= 0 && t < rw.aux) ? rw.src + (int64_t)t * d_in : -1;
  } else {
    src = rows[r].src;
  }
  float v[E];
  if (src < 0) {
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = (c0 + j < d_in) ? pad : 0.f;
  } else if (src + d_in > dense_len) {
    *err = 1;
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = 0.f;
  } else if ((d_in & 3) == 0 && (src & 3) == 0) {
#pragma unroll
    for (int h = 0; h < E; h += 4) {
      if (c0 + h < d_in) {  // d_in % 4 == 0: all 4 columns are inputs
        const float4 a = *(const float4*)(dense + src + c0 + h);
        v[h + 0] = a.x; v[h + 1] = a.y; v[h + 2] = a.z; v[h + 3] = a.w;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[h + j] = 0.f;
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = (c0 + j < d_in) ? dense[src + c0 + j] : 0.f;
  }
  if (BF16) {
    bf16_t* y = (bf16_t*)X + r * ldx + c0;
    *(uint4*)y = make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7]));
  } else {
    float* y = (float*)X + r * ldx + c0;
#pragma unroll
    for (int h = 0; h < E; h += 4) *(float4*)(y + h) = make_float4(v[h], v[h + 1], v[h + 2], v[h + 3]);
  }
}

// ---------------------------------------------------------------- embedding bags

constexpr int EMB_DIM = 64;       // one table row = 128 bytes of bf16
constexpr int MAX_TABLES = 64;
constexpr int EMB_CHUNK = 8;      // ids loaded (one per lane of a group) per round

// One 8-lane group per bag; lane l8 owns dims [8 l8, 8 l8 + 8) of the 64-dim
// table rows. The grid is table-major: workgroups [t nrb, (t + 1) nrb) serve
// table t for 32 ROUNDS consecutive rows each, so at any time the whole chip
// gathers from one or two tables and every XCD's L2 and the Infinity Cache
// hold their hot rows (all tables at once per row measured 1.5x slower, 4 or 8
// tables 1.2x slower).
//
// The kernel is bound by its chains of dependent loads and its instructions
// before memory: with every id the same row (all gathers in L1) a workgroup per
// 32 bags, ranked through LDS, took 104 us of the 140 us it took on Zipf ids
// (32768 rows x 26 bags of 1..20 ids; 64 bytes a clock and compute unit, what L1
// and L2 return to 32 waves of 8 gathers each, would be 37 us). Now 105 us on
// Zipf ids and 63 us on one row, at 7 waves per SIMD (72 registers; at 5 waves
// 115 us).
// A wave takes the bags of 8 ROUNDS rows, bag i in lane i first:
//  - a bag's place among its row's ids comes from the routing step (`ends`:
//    two loads per bag; without it, with 8 bags a wave, from an 8-lane sum of
//    the preceding bag lengths);
//  - the lanes rank the bags by length (six ballots on a capped key) and the
//    wave walks 8 of them at a time, longest first: the bags of a round then have
//    similar lengths, and the longest bounds the round's loop;
//  - lane i of a group loads and checks id c + i of a chunk and turns it into a
//    byte offset into the table, out of range for an id that is invalid or past
//    the bag; the offset is broadcast and a buffer load returns zeros for it
//    (BIG: tables of 4 GiB or more, with 64-bit addresses and a predicate). The
//    next chunk's or round's ids load during a chunk's gathers;
//  - a chunk that the longest bag ends in gathers 4, 2 and 1 ids.
// Sums are fp32 in id order (a fixed order that depends on the bag only),
// stored as bf16. The workgroups of table 0 also write the rows' dense features
// and zero tails. Reads stay inside the ids arena and the tables: an id
// position outside the arena or an id outside its table sets *err = 1 and
// contributes nothing.
template <int ROUNDS, bool BIG>
__global__ __launch_bounds__(256, ROUNDS == 1 ? 8 : 7) void k_embbag(const rb_k_row* __restrict__ rows, int n_rows,
                                                   const int32_t* __restrict__ lens,
                                                   const int32_t* __restrict__ ends,
                                                   const int32_t* __restrict__ ids, int64_t ids_len,
                                                   const bf16_t* const* __restrict__ tables, int n_tables,
                                                   int64_t table_rows, const float* __restrict__ dense,
                                                   int n_dense, bf16_t* __restrict__ X, int ldx, float pad,
                                                   int* __restrict__ err) {
  constexpr int NB = 8 * ROUNDS;         // bags per wave
  const int nrb = gridDim.x / n_tables;  // row blocks per table
  const int t = blockIdx.x / nrb;
  const int rb0 = (blockIdx.x - t * nrb) * 4 * NB;  // the workgroup's first row
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 3, l8 = lane & 7;
  const int r0 = __builtin_amdgcn_readfirstlane(rb0 + (tid >> 6) * NB);
  auto from = [](int v, int src_lane) { return __builtin_amdgcn_ds_bpermute(src_lane * 4, v); };
  // a position in the ids arena (one outside it stays outside for the whole bag)
  typedef typename std::conditional<BIG, int64_t, uint32_t>::type pos_t;
  const pos_t n_ids = (pos_t)ids_len;
  auto to_pos = [&](int64_t p) { return BIG ? (pos_t)p : (p >= 0 && p <= ids_len ? (pos_t)p : (pos_t)n_ids); };
  // 1. lane i: bag i's length (-1: no bag, -2: a padding row) and its first
  //    id's position in the ids arena
  int L = -1;
  pos_t pos = 0;
  if (ROUNDS > 1 || ends) {
    if (lane < NB && r0 + lane < n_rows) {
      const int row = r0 + lane;
      const int e1 = ends[(int64_t)t * n_rows + row], e0 = t ? ends[(int64_t)(t - 1) * n_rows + row] : 0;
      const int64_t src = rows[row].src, aux = rows[row].aux;
      L = src < 0 ? -2 : e1 - e0;
      pos = to_pos(aux + e0);
    }
  } else {
    int len = -1;
    pos_t p = 0;
    if (r0 + g < n_rows) {
      const rb_k_row rw = rows[r0 + g];
      if (rw.src < 0) {
        len = -2;
      } else {
        // lane l8 loads the lengths of tables l8, l8 + 8, ... below t and the
        // bag's own length, all issued before any is used
        int v[MAX_TABLES / 8];
#pragma unroll
        for (int u = 0; u < MAX_TABLES / 8; ++u) {
          const int f = l8 + 8 * u;
          v[u] = f < t ? lens[rw.lens + f] : 0;
        }
        len = lens[rw.lens + t];
        int pre = 0;
#pragma unroll
        for (int u = 0; u < MAX_TABLES / 8; ++u) pre += v[u];
        pre += __shfl_xor(pre, 1);
        pre += __shfl_xor(pre, 2);
        pre += __shfl_xor(pre, 4);
        p = to_pos(rw.aux + pre);
      }
    }
    const int a = __shfl(len, l8 * 8);
    const pos_t b = __shfl(p, l8 * 8);
    if (g == 0) {
      L = a;
      pos = b;
    }
  }
  // 2. ranked longest first (ties by row; lengths past 60 count as equal): bag
  //    of rank p in lane p
  int row_of = lane;
  if (ROUNDS > 1) {
    const int key = min(L, 60) + 2;
    uint32_t gt = 0, eq = NB < 32 ? (1u << (NB & 31)) - 1u : 0xffffffffu;
#pragma unroll
    for (int bit = 5; bit >= 0; --bit) {
      const bool one = (key >> bit) & 1;
      const uint32_t b = (uint32_t)__ballot(one);
      if (!one) gt |= eq & b;
      eq &= one ? b : ~b;
    }
    const int to = 4 * (lane < NB ? __popc(gt) + __popc(eq & ((1u << (lane & 31)) - 1u)) : lane);
    L = __builtin_amdgcn_ds_permute(to, L);
    row_of = __builtin_amdgcn_ds_permute(to, lane);
    if constexpr (BIG)
      pos = (pos_t)(((uint64_t)(uint32_t)__builtin_amdgcn_ds_permute(to, (int)((uint64_t)pos >> 32)) << 32) |
                    (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(uint32_t)pos));
    else
      pos = (pos_t)__builtin_amdgcn_ds_permute(to, (int)pos);
  }
  // 3. the walks
  const bf16_t* tab = tables[t];
  constexpr uint32_t NONE = 0xffffff00u;  // past every table that is not BIG
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)tab, 0, BIG ? 0 : (int)(uint32_t)(table_rows * EMB_DIM * 2),
                                                      0x00020000);
  const auto irsrc = __builtin_amdgcn_make_buffer_rsrc((void*)ids, 0, BIG ? 0 : (int)(uint32_t)(ids_len * 4), 0x00020000);
  const int gsel = (lane & ~7) * 4;  // this group's first lane, as a permute address
  // this lane's id of chunk c of a bag as a byte offset into the table (BIG:
  // the id, or -1)
  auto chunk_off = [&](int bL, pos_t bpos, int c) -> uint32_t {
    const int j = c + l8;
    uint32_t o = BIG ? 0xffffffffu : NONE;
    if (j < bL) {
      const pos_t p = bpos + (pos_t)j;
      int id = -1;
      if constexpr (BIG) {
        if (p >= 0 && p < n_ids) id = ids[p];
      } else {
        if (p < n_ids) id = (int)__builtin_amdgcn_raw_buffer_load_b32(irsrc, (int)(p * 4), 0, 0);
      }
      if (BIG ? (uint64_t)(int64_t)id < (uint64_t)table_rows : (uint32_t)id < (uint32_t)table_rows)
        o = BIG ? (uint32_t)id : (uint32_t)id * (EMB_DIM * 2);
      else
        *err = 1;
    }
    return o;
  };
  int bL = __shfl(L, g);
  pos_t bpos = __shfl(pos, g);
  uint32_t nxt = chunk_off(bL, bpos, 0);
  for (int i = 0; i < ROUNDS; ++i) {
    int Lw = bL;  // the round's longest bag
    Lw = max(Lw, __shfl_xor(Lw, 8));
    Lw = max(Lw, __shfl_xor(Lw, 16));
    Lw = __builtin_amdgcn_readfirstlane(max(Lw, __shfl_xor(Lw, 32)));
    const int brow = from(row_of, i * 8 + g), myL = bL;
    float acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.f;
    auto gather = [&](auto nc, uint32_t my, int u0) {  // ids u0 .. u0 + n - 1 of a chunk
      constexpr int n = decltype(nc)::value;
      u32x4_t q[n];
#pragma unroll
      for (int u = 0; u < n; ++u) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_ds_bpermute(gsel + (u0 + u) * 4, (int)my);
        if constexpr (BIG) {
          q[u] = (u32x4_t){0u, 0u, 0u, 0u};
          if (o != 0xffffffffu) q[u] = *(const u32x4_t*)((const char*)tab + (int64_t)o * (EMB_DIM * 2) + l8 * 16);
        } else {
          q[u] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(o + l8 * 16), 0, 0));
        }
      }
#pragma unroll
      for (int u = 0; u < n; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          acc[2 * k] += __uint_as_float(q[u][k] << 16);
          acc[2 * k + 1] += __uint_as_float(q[u][k] & 0xffff0000u);
        }
    };
    int c = 0;
    do {
      const uint32_t my = nxt;
      const int rem = Lw - c;  // uniform
      c += EMB_CHUNK;
      if (rem <= EMB_CHUNK) {  // on to the next round's bag (after the last round: none)
        bL = i + 1 < ROUNDS ? __shfl(L, i * 8 + 8 + g) : -1;
        bpos = __shfl(pos, i * 8 + 8 + g);
      }
      nxt = chunk_off(bL, bpos, rem <= EMB_CHUNK ? 0 : c);
      if (rem >= EMB_CHUNK) {
        gather(ic<8>{}, my, 0);
      } else if (rem > 0) {
        if (rem & 4) gather(ic<4>{}, my, 0);
        if (rem & 2) gather(ic<2>{}, my, rem & 4);
        if (rem & 1) gather(ic<1>{}, my, rem & 6);
      }
    } while (c < Lw);
    if (myL != -1) {
      u32x4_t o = {pack2_rne(acc[0], acc[1]), pack2_rne(acc[2], acc[3]), pack2_rne(acc[4], acc[5]),
                   pack2_rne(acc[6], acc[7])};
      if (myL == -2) {
        const uint32_t p = f2bf(pad);
        o = (u32x4_t){p | (p << 16), p | (p << 16), p | (p << 16), p | (p << 16)};
      }
      *(u32x4_t*)(X + (int64_t)(r0 + brow) * ldx + t * EMB_DIM + l8 * 8) = o;
    }
  }
  if (t == 0) {
    // the dense features and zero tail (columns n_tables EMB_DIM .. ldx, a multiple of 8
    // wide): one 8-column chunk, a 16-byte store, per thread and pass, so that
    // the loads of all the block's rows are in flight at once
    const int demb = n_tables * EMB_DIM, cpr = (ldx - demb) >> 3;
    for (int e = tid; e < 4 * NB * cpr; e += 256) {
      const int i = e / cpr, c = e - i * cpr;
      if (rb0 + i >= n_rows) break;
      const rb_k_row rw = rows[rb0 + i];
      uint32_t h[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int d = 8 * c + k;
        h[k] = d < n_dense ? (uint32_t)f2bf(rw.src < 0 ? pad : dense[rw.src + d]) : 0u;
      }
      const u32x4_t o = {h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
      *(u32x4_t*)(X + (int64_t)(rb0 + i) * ldx + demb + 8 * c) = o;
    }
  }
}

// Embedding bags with the ids of a batch block deduplicated per table
// (compressing away features common to a batch of examples, paper section
// 2.2): workgroup (table t, block of DD_ROWS rows) stages the block's bag ids
// for table t in LDS, finds the distinct ones with an open-addressing hash in
// LDS, gathers each distinct table row once into LDS (up to DD_UCAP rows,
// 128 bytes each, 16-byte loads by 8-lane groups), then sums every bag from
// LDS in id order. The sums are the same fp32 additions in the same order as
// k_embbag's, so the outputs are bit-identical; only the table rows gathered
// per block change (measured on the ranking workload: 672 ids per 64-row block
// and table, 345 distinct). Ids past DD_NMAX positions in the block, or
// distinct rows past DD_UCAP, are gathered from the table directly. The same
// bounds as k_embbag: an id position outside the ids arena or an id outside its
// table sets *err = 1 and contributes +0.
constexpr int DD_ROWS = 64;     // rows per workgroup
constexpr int DD_NT = 512;      // threads per workgroup: 8 per row, 64 8-lane groups
constexpr int DD_NMAX = 1280;   // id positions staged per workgroup (64 rows x 20 ids)
constexpr int DD_HS = 2048;     // hash slots (> DD_NMAX: an insert always finds a free slot)
constexpr int DD_UCAP = 448;    // distinct table rows staged per workgroup (56 KB)

__global__ __launch_bounds__(DD_NT) void k_embbag_dedup(const rb_k_row* __restrict__ rows, int n_rows,
                                                        const int32_t* __restrict__ lens,
                                                        const int32_t* __restrict__ ids, int64_t ids_len,
                                                        const bf16_t* const* __restrict__ tables, int n_tables,
                                                        int64_t table_rows, const float* __restrict__ dense,
                                                        int n_dense, bf16_t* __restrict__ X, int ldx, float pad,
                                                        int* __restrict__ err) {
  __shared__ u32x4_t s_u[DD_UCAP][8];   // distinct table rows (8 x 16 bytes each)
  __shared__ int32_t s_key[DD_HS];      // hash slot -> table row id (-1: empty)
  __shared__ int16_t s_slot[DD_HS];     // hash slot -> distinct-row index
  __shared__ int32_t s_ids[DD_NMAX];    // the block's ids, bag after bag (-1: invalid)
  __shared__ int16_t s_k[DD_NMAX];      // id position -> hash slot, then -> distinct-row index (-1: invalid)
  __shared__ int32_t s_uid[DD_UCAP];    // distinct-row index -> table row id
  __shared__ int32_t s_len[DD_ROWS], s_start[DD_ROWS + 1];
  __shared__ int64_t s_id0[DD_ROWS];    // a row's first id of table t in the ids arena
  __shared__ int s_wsum[DD_NT / 64];
  const int nrb = gridDim.x / n_tables;
  const int t = blockIdx.x / nrb;
  const int r0 = (blockIdx.x - t * nrb) * DD_ROWS;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int g = tid >> 3, l8 = tid & 7;  // 8-lane group g serves row g
  const bf16_t* tab = tables[t];
  for (int h = tid; h < DD_HS; h += DD_NT) s_key[h] = -1;
  // 1. row g's bag of table t: its 8 lanes load the row's bag lengths
  //    (lane l8 those of tables l8, l8 + 8, ... below t, all at once) and sum
  //    them; then an exclusive scan over the block's rows
  {
    int pre = 0, L = 0;
    int64_t aux = 0;
    bool real = false;
    if (r0 + g < n_rows) {
      const rb_k_row rw = rows[r0 + g];
      real = rw.src >= 0;
      if (real) {
        int v[MAX_TABLES / 8];
#pragma unroll
        for (int u = 0; u < MAX_TABLES / 8; ++u) {
          const int f = l8 + 8 * u;
          v[u] = f < t ? lens[rw.lens + f] : 0;
        }
#pragma unroll
        for (int u = 0; u < MAX_TABLES / 8; ++u) pre += v[u];
        L = lens[rw.lens + t];
        aux = rw.aux;
      }
    }
    pre += __shfl_xor(pre, 1);
    pre += __shfl_xor(pre, 2);
    pre += __shfl_xor(pre, 4);
    if (l8 == 0) {
      s_len[g] = real ? max(L, 0) : 0;
      s_id0[g] = aux + pre;
    }
  }
  __syncthreads();
  if (wid == 0) {  // exclusive scan of the 64 bag lengths
    const int v = s_len[lane];
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(incl, o);
      if (lane >= o) incl += u;
    }
    s_start[lane] = incl - v;
    if (lane == 63) s_start[DD_ROWS] = incl;
  }
  __syncthreads();
  const int n_pos = min(s_start[DD_ROWS], DD_NMAX);
  // 2. stage the ids: row g's 8 lanes take its bag's positions l8, l8 + 8, ...
  {
    const int L = s_len[g], st = s_start[g];
    const int64_t id0 = s_id0[g];
    for (int j0 = 0; j0 < L && st + j0 < DD_NMAX; j0 += 32) {
      int v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j0 + l8 + 8 * u;
        const int64_t pos = id0 + j;
        v[u] = (j < L && pos >= 0 && pos < ids_len) ? ids[pos] : -1;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j0 + l8 + 8 * u;
        if (j < L && st + j < DD_NMAX) {
          int id = v[u];
          if ((uint64_t)(int64_t)id >= (uint64_t)table_rows) {
            *err = 1;
            id = -1;
          }
          s_ids[st + j] = id;
        }
      }
    }
  }
  __syncthreads();
  // 3. distinct ids: insert every staged id into the hash (linear probing)
  for (int i = tid; i < n_pos; i += DD_NT) {
    const int id = s_ids[i];
    int h = -1;
    if (id >= 0) {
      h = (int)(((uint32_t)id * 2654435761u) >> 21);  // 11 bits: DD_HS slots
      for (;;) {
        const int old = atomicCAS(&s_key[h], -1, id);
        if (old == -1 || old == id) break;
        h = (h + 1) & (DD_HS - 1);
      }
    }
    s_k[i] = (int16_t)h;
  }
  __syncthreads();
  // 4. number the occupied slots (block scan, 4 slots per thread)
  {
    constexpr int SPT = DD_HS / DD_NT;
    int occ[SPT], c = 0;
#pragma unroll
    for (int k = 0; k < SPT; ++k) {
      occ[k] = s_key[tid * SPT + k] >= 0;
      c += occ[k];
    }
    int incl = c;
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(incl, o);
      if (lane >= o) incl += u;
    }
    if (lane == 63) s_wsum[wid] = incl;
    __syncthreads();
    int base = incl - c;
    for (int w = 0; w < wid; ++w) base += s_wsum[w];
#pragma unroll
    for (int k = 0; k < SPT; ++k) {
      if (occ[k]) {
        s_slot[tid * SPT + k] = (int16_t)base;
        if (base < DD_UCAP) s_uid[base] = s_key[tid * SPT + k];
        ++base;
      }
    }
  }
  __syncthreads();
  int n_all = 0;
#pragma unroll
  for (int w = 0; w < DD_NT / 64; ++w) n_all += s_wsum[w];
  const int n_u = min(n_all, DD_UCAP);
  // 5. every distinct row once (8-lane group g: rows g, g + 64, ...), and each
  //    staged position's distinct-row index (hash slot replaced by it)
  {
    constexpr int UNR = 4;
    for (int k0 = g; k0 < n_u; k0 += (DD_NT / 8) * UNR) {
      u32x4_t v[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int k = k0 + (DD_NT / 8) * u;
        if (k < n_u) v[u] = *(const u32x4_t*)(tab + (int64_t)s_uid[k] * EMB_DIM + l8 * 8);
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int k = k0 + (DD_NT / 8) * u;
        if (k < n_u) s_u[k][l8] = v[u];
      }
    }
    for (int i = tid; i < n_pos; i += DD_NT) {
      const int h = s_k[i];
      // rows past the staged ones keep -2 - hash slot: gathered directly
      s_k[i] = (int16_t)(h < 0 ? -1 : (s_slot[h] < DD_UCAP ? s_slot[h] : -2 - h));
    }
  }
  __syncthreads();
  // 6. row g's bag from the staged rows, in id order (fp32), stored as bf16;
  //    8 ids per round, their reads issued before any is added
  if (r0 + g < n_rows) {
    const rb_k_row rw = rows[r0 + g];
    u32x4_t o;
    if (rw.src < 0) {
      const uint32_t pv = f2bf(pad);
      o = (u32x4_t){pv | (pv << 16), pv | (pv << 16), pv | (pv << 16), pv | (pv << 16)};
    } else {
      float acc[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] = 0.f;
      const int L = s_len[g], st = s_start[g];
      for (int j0 = 0; j0 < L; j0 += 8) {
        u32x4_t q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int j = j0 + u, i = st + j;
          q[u] = (u32x4_t){0u, 0u, 0u, 0u};
          if (j < L) {
            if (i < DD_NMAX) {
              const int k = s_k[i];
              if (k >= 0)
                q[u] = s_u[k][l8];
              else if (k <= -2)
                q[u] = *(const u32x4_t*)(tab + (int64_t)s_key[-2 - k] * EMB_DIM + l8 * 8);
            } else {  // past the staged positions: straight from the arena and the table
              const int64_t pos = s_id0[g] + j;
              const int id = (pos >= 0 && pos < ids_len) ? ids[pos] : -1;
              if ((uint64_t)(int64_t)id < (uint64_t)table_rows)
                q[u] = *(const u32x4_t*)(tab + (int64_t)id * EMB_DIM + l8 * 8);
              else
                *err = 1;
            }
          }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if (j0 + u < L) {
            acc[0] += bf2f(q[u].x & 0xffffu); acc[1] += bf2f(q[u].x >> 16);
            acc[2] += bf2f(q[u].y & 0xffffu); acc[3] += bf2f(q[u].y >> 16);
            acc[4] += bf2f(q[u].z & 0xffffu); acc[5] += bf2f(q[u].z >> 16);
            acc[6] += bf2f(q[u].w & 0xffffu); acc[7] += bf2f(q[u].w >> 16);
          }
        }
      }
      o.x = pack2(acc[0], acc[1]);
      o.y = pack2(acc[2], acc[3]);
      o.z = pack2(acc[4], acc[5]);
      o.w = pack2(acc[6], acc[7]);
    }
    *(u32x4_t*)(X + (int64_t)(r0 + g) * ldx + t * EMB_DIM + l8 * 8) = o;
  }
  // the workgroups of table 0 also write the rows' dense features and zero tails
  if (t == 0) {
    const int demb = n_tables * EMB_DIM;
    for (int i = 0; i < DD_ROWS && r0 + i < n_rows; ++i) {
      const rb_k_row rw = rows[r0 + i];
      bf16_t* xr = X + (int64_t)(r0 + i) * ldx;
      for (int c = demb + tid; c < ldx; c += DD_NT) {
        const int d = c - demb;
        xr[c] = d < n_dense ? f2bf(rw.src < 0 ? pad : dense[rw.src + d]) : (bf16_t)0;
      }
    }
  }
}

// The arena offset of every packed token row, one wave per sequence slot:
// token t of slot e is packed row rows[e].lens + t and starts at element
// rows[e].src + t d_in of the dense arena. The checks are k_assemble_seq's; a
// sequence that fails them sets *err and leaves its entries as they are (the
// layer that reads them checks each against the arena).
__global__ __launch_bounds__(256) void k_token_rows(const rb_k_row* __restrict__ rows, int n_slots, int T,
                                                    int64_t dense_len, int d_in, int64_t* __restrict__ src,
                                                    int64_t n_src, int* __restrict__ err) {
  const int e = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (e >= n_slots) return;
  const rb_k_row rw = rows[e];
  if (rw.src < 0 || rw.aux <= 0) return;
  const int64_t L = rw.aux;
  if (L > T || rw.src + L * d_in > dense_len || rw.lens < 0 || rw.lens + L > n_src) {
    if ((threadIdx.x & 63) == 0) *err = 1;
    return;
  }
  for (int t = threadIdx.x & 63; t < L; t += 64) src[rw.lens + t] = rw.src + (int64_t)t * d_in;
}

// ---------------------------------------------------------------- heads and split

// 16 lanes per row (16 rows per workgroup): a K-long dot product, each lane
// taking 8 consecutive elements of every 128 with 16-byte loads (or every
// 16th element when rows are not 16-byte aligned), a 16-lane butterfly, bias,
// activation, and the store into the request's output row (one wave per row
// with 2-byte loads measured 1.5x slower on 256-wide rows).
template <int ACT>
__global__ __launch_bounds__(256) void k_head(const rb_k_row* __restrict__ rows, int n,
                                              const bf16_t* __restrict__ H, int ldh,
                                              const bf16_t* __restrict__ w, float b, int K, int vec,
                                              float* __restrict__ out) {
  const int r = blockIdx.x * 16 + (threadIdx.x >> 4), l = threadIdx.x & 15;
  float s = 0.f;
  int64_t o = -1;
  if (r < n) {
    o = rows[r].out;
    if (o >= 0) {
      const bf16_t* h = H + (int64_t)r * ldh;
      if (vec) {
        for (int k = l * 8; k < K; k += 128) {
          const u32x4_t hv = *(const u32x4_t*)(h + k), wv = *(const u32x4_t*)(w + k);
          s += bf2f(hv.x & 0xffffu) * bf2f(wv.x & 0xffffu);
          s += bf2f(hv.x >> 16) * bf2f(wv.x >> 16);
          s += bf2f(hv.y & 0xffffu) * bf2f(wv.y & 0xffffu);
          s += bf2f(hv.y >> 16) * bf2f(wv.y >> 16);
          s += bf2f(hv.z & 0xffffu) * bf2f(wv.z & 0xffffu);
          s += bf2f(hv.z >> 16) * bf2f(wv.z >> 16);
          s += bf2f(hv.w & 0xffffu) * bf2f(wv.w & 0xffffu);
          s += bf2f(hv.w >> 16) * bf2f(wv.w >> 16);
        }
      } else {
        for (int k = l; k < K; k += 16) s += bf2f(h[k]) * bf2f(w[k]);
      }
    }
  }
  // 16-lane sum: every lane of the wave takes part in the exchanges
  s += __shfl_xor(s, 1);
  s += __shfl_xor(s, 2);
  s += __shfl_xor(s, 4);
  s += __shfl_xor(s, 8);
  if (l == 0 && o >= 0) out[o] = act_fn<ACT>(s + b);
}

// ---------------------------------------------------------------- fused MLP tail

// The last two hidden layers (ReLU, N2 = 512 then N3 = 256 outputs) and the
// narrow head of a bf16 model, fused per block of MT_BM rows: the first layer's
// k-steps stream H1 rows and W2 rows through two LDS stages; its outputs
// (bias, ReLU, bf16) stay in LDS as the second layer's input while W3 streams
// through two more stages; the second layer's outputs (bias, ReLU, bf16) go to
// LDS and the head reads them there. Each output is accumulated in the same k
// order with the same 16x16x32 bf16 MFMA as k_gemm_bf16, rounded the same way,
// and the head sums exactly as k_head does (16 lanes per row, 8 consecutive
// elements of every 128 per lane, then a 16-lane butterfly), so the results
// are bit-identical to running the two layers and the head separately; only
// the two hidden layers' round trips through memory and two launches go away.
// 8 waves: 2 x 4 over the 128 x 512 tile of the first layer (64 x 128 each),
// 2 x 4 over the 128 x 256 tile of the second (64 x 64 each). Operand rows of
// 64 bytes per k-step sit in LDS with their four 16-byte chunks permuted by
// row, and the 1024-byte rows of the first layer's output with their 64 chunks
// permuted by row, so that a fragment read's 32 rows spread over the banks.
constexpr int MT_BM = 128, MT_NT = 512, MT_N2 = 512, MT_N3 = 256, MT_KS = 32;
constexpr int MT_A_BYTES = MT_BM * 64, MT_B_BYTES = MT_N2 * 64;           // one stage of the first layer
constexpr int MT_Y2 = 0;                                                // [MT_BM][MT_N2] bf16, 128 KB
constexpr int MT_W3 = MT_BM * MT_N2 * 2;                                // two stages of [MT_N3][64 B]
constexpr int MT_LDS = MT_W3 + 2 * MT_N3 * 64;                          // 160 KB
static_assert(2 * (MT_A_BYTES + MT_B_BYTES) <= MT_W3, "first-layer stages fit below the W3 stages");

__device__ __forceinline__ uint32_t mt_addr4(int row, int c) { return (uint32_t)(row * 64 + ((c ^ ((row >> 2) & 3)) << 4)); }
__device__ __forceinline__ uint32_t mt_addr_y2(int row, int c) { return (uint32_t)(row * 1024 + ((c ^ (row & 63)) << 4)); }

template <int ACT>
__global__ __launch_bounds__(MT_NT) void k_mlp_tail(const bf16_t* __restrict__ H1, int ldh1, int K2,
                                                    const bf16_t* __restrict__ W2, int ldw2,
                                                    const float* __restrict__ b2, const bf16_t* __restrict__ W3,
                                                    int ldw3, const float* __restrict__ b3,
                                                    const bf16_t* __restrict__ w4, float b4,
                                                    const rb_k_row* __restrict__ rows, int M,
                                                    float* __restrict__ out) {
  __shared__ __align__(16) unsigned char lds[MT_LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wid >> 2, wn = wid & 3;
  const int m0 = blockIdx.x * MT_BM;
  const int lrow = tid >> 2, lc = tid & 3;  // the row (of 128) and chunk this thread loads
  // ---- first layer: Y2 = relu(H1 W2^T + b2) on rows [m0, m0 + 128)
  const bf16_t* a_src = H1 + (int64_t)(m0 + min(lrow, M - 1 - m0)) * ldh1 + lc * 8;  // rows past M: a copy
  // k-step operands go global -> registers -> LDS, loaded two k-steps ahead
  // into two register sets (the k loops are unrolled by two so that each set
  // stays in registers)
  struct Op1 {
    u32x4_t a, b[4];
  };
  auto load1 = [&](Op1& r, int kt) {
    const int k0 = kt * MT_KS;
    r.a = *(const u32x4_t*)(a_src + k0);
#pragma unroll
    for (int i = 0; i < 4; ++i) r.b[i] = *(const u32x4_t*)(W2 + (int64_t)(lrow + 128 * i) * ldw2 + k0 + lc * 8);
  };
  auto store1 = [&](const Op1& r, int st) {
    unsigned char* base = lds + st * (MT_A_BYTES + MT_B_BYTES);
    *(u32x4_t*)(base + mt_addr4(lrow, lc)) = r.a;
#pragma unroll
    for (int i = 0; i < 4; ++i) *(u32x4_t*)(base + MT_A_BYTES + mt_addr4(lrow + 128 * i, lc)) = r.b[i];
  };
  floatx4_t acc[4][8];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
  auto mma1 = [&](int st) {  // lane l holds row l % 16, chunk l / 16
    const unsigned char* base = lds + st * (MT_A_BYTES + MT_B_BYTES);
    u32x4_t fa[4], fb[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) fa[i] = *(const u32x4_t*)(base + mt_addr4(wm * 64 + i * 16 + (lane & 15), lane >> 4));
#pragma unroll
    for (int j = 0; j < 8; ++j)
      fb[j] = *(const u32x4_t*)(base + MT_A_BYTES + mt_addr4(wn * 128 + j * 16 + (lane & 15), lane >> 4));
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fa[i]),
                                                            __builtin_bit_cast(bf16x8_t, fb[j]), acc[i][j], 0, 0, 0);
  };
  // k-step kt: load kt + 2 into the set kt held, multiply stage kt % 2, store
  // kt + 1 (loaded a k-step ago) into the other stage
  auto step1 = [&](int kt, int nk, Op1& mine, Op1& next) {
    if (kt + 2 < nk) load1(mine, kt + 2);
    mma1(kt & 1);
    if (kt + 1 < nk) store1(next, (kt + 1) & 1);
    __syncthreads();
  };
  const int nk = K2 / MT_KS;
  Op1 r0, r1;
  load1(r0, 0);
  if (nk > 1) load1(r1, 1);
  store1(r0, 0);
  __syncthreads();
  for (int kt = 0; kt < nk; kt += 2) {
    step1(kt, nk, r0, r1);
    if (kt + 1 < nk) step1(kt + 1, nk, r1, r0);
  }
  // W3's first two k-steps load while the first layer's outputs go to LDS
  struct Op2 {
    u32x4_t b[2];
  };
  auto load2 = [&](Op2& r, int kt) {
    const int k0 = kt * MT_KS;
#pragma unroll
    for (int i = 0; i < 2; ++i) r.b[i] = *(const u32x4_t*)(W3 + (int64_t)(lrow + 128 * i) * ldw3 + k0 + lc * 8);
  };
  auto store2 = [&](const Op2& r, int st) {
    unsigned char* base = lds + MT_W3 + st * (MT_N3 * 64);
#pragma unroll
    for (int i = 0; i < 2; ++i) *(u32x4_t*)(base + mt_addr4(lrow + 128 * i, lc)) = r.b[i];
  };
  Op2 w0, w1;
  load2(w0, 0);
  load2(w1, 1);
  // accumulator (i, j) register r of lane l: row 4 (l / 16) + r, column l % 16
  // of its 16 x 16 block; bias and ReLU per column, then each group of four rows
  // transposed across the quad so a lane holds four consecutive columns of one
  // row, rounded to bf16 as k_gemm_bf16's epilogue rounds
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int col0 = wn * 128 + j * 16;
    const float bb = b2[col0 + (lane & 15)];
    const int colq = col0 + (lane & 12);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float q[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) q[k] = act_fn<RB_ACT_RELU>(acc[i][j][k] + bb);
      quad_transpose4(q, lane);
      const int row = wm * 64 + i * 16 + 4 * (lane >> 4) + (lane & 3);
      const u32x2_t o = {pack2_rne(q[0], q[1]), pack2_rne(q[2], q[3])};
      *(u32x2_t*)(lds + MT_Y2 + mt_addr_y2(row, colq >> 3) + ((colq & 4) ? 8 : 0)) = o;
    }
  }
  store2(w0, 0);
  __syncthreads();
  // ---- second layer: Y3 = relu(Y2 W3^T + b3)
  floatx4_t acc3[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc3[i][j][r] = 0.f;
  auto mma2 = [&](int kt) {
    const unsigned char* base = lds + MT_W3 + (kt & 1) * (MT_N3 * 64);
    u32x4_t fa[4], fb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = wm * 64 + i * 16 + (lane & 15);
      fa[i] = *(const u32x4_t*)(lds + MT_Y2 + mt_addr_y2(row, kt * 4 + (lane >> 4)));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      fb[j] = *(const u32x4_t*)(base + mt_addr4(wn * 64 + j * 16 + (lane & 15), lane >> 4));
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc3[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fa[i]),
                                                             __builtin_bit_cast(bf16x8_t, fb[j]), acc3[i][j], 0, 0, 0);
  };
  constexpr int nk3 = MT_N2 / MT_KS;
  auto step2 = [&](int kt, Op2& mine, Op2& next) {
    if (kt + 2 < nk3) load2(mine, kt + 2);
    mma2(kt);
    if (kt + 1 < nk3) store2(next, (kt + 1) & 1);
    __syncthreads();
  };
  for (int kt = 0; kt < nk3; kt += 2) {
    step2(kt, w0, w1);
    step2(kt + 1, w1, w0);
  }
  // Y3 (bias, ReLU, bf16) to LDS, row-major [MT_BM][MT_N3] over the first
  // layer's outputs (no longer read)
  unsigned char* y3 = lds;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int col0 = wn * 64 + j * 16;
    const float bb = b3[col0 + (lane & 15)];
    const int colq = col0 + (lane & 12);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float q[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) q[k] = act_fn<RB_ACT_RELU>(acc3[i][j][k] + bb);
      quad_transpose4(q, lane);
      const int row = wm * 64 + i * 16 + 4 * (lane >> 4) + (lane & 3);
      const u32x2_t o = {pack2_rne(q[0], q[1]), pack2_rne(q[2], q[3])};
      *(u32x2_t*)(y3 + row * (MT_N3 * 2) + colq * 2) = o;
    }
  }
  __syncthreads();
  // ---- head, as k_head: 16 lanes per row, lane l taking elements
  // [8 l + 128 i, 8 l + 128 i + 8), then a 16-lane butterfly
  const int l16 = tid & 15;
#pragma unroll
  for (int pass = 0; pass < MT_BM / (MT_NT / 16); ++pass) {
    const int row = pass * (MT_NT / 16) + (tid >> 4);
    float s = 0.f;
    for (int k = l16 * 8; k < MT_N3; k += 128) {
      const u32x4_t hv = *(const u32x4_t*)(y3 + row * (MT_N3 * 2) + k * 2), wv = *(const u32x4_t*)(w4 + k);
      s += bf2f(hv.x & 0xffffu) * bf2f(wv.x & 0xffffu);
      s += bf2f(hv.x >> 16) * bf2f(wv.x >> 16);
      s += bf2f(hv.y & 0xffffu) * bf2f(wv.y & 0xffffu);
      s += bf2f(hv.y >> 16) * bf2f(wv.y >> 16);
      s += bf2f(hv.z & 0xffffu) * bf2f(wv.z & 0xffffu);
      s += bf2f(hv.z >> 16) * bf2f(wv.z >> 16);
      s += bf2f(hv.w & 0xffffu) * bf2f(wv.w & 0xffffu);
      s += bf2f(hv.w >> 16) * bf2f(wv.w >> 16);
    }
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    s += __shfl_xor(s, 4);
    s += __shfl_xor(s, 8);
    if (l16 == 0 && m0 + row < M) {
      const int64_t o = rows[m0 + row].out;
      if (o >= 0) out[o] = act_fn<ACT>(s + b4);
    }
  }
}

constexpr int POOL_MAX_D = 1024, POOL_MAX_OUT = 16;

// One workgroup per sequence slot. The slot's real tokens are summed in P
// consecutive parts (part p: tokens [p L / P, (p + 1) L / P); tokens past L are
// never read, so padding cannot reach the mean), each in token order; the
// partial sums are added in part order and divided by L: a fixed order, and P
// depends on L only (4 up to POOL_SHORT tokens, else 16), so the result depends
// on the sequence only, not on NW nor on its slot's length. A wave sums P / NW
// parts side by side, each lane owning float4 columns, with 8 token loads (4 of
// a short sequence) in flight; a launch waits for one wave's chain of round
// trips, so 16 waves take a long sequence when there are few, and 4 otherwise.
// Back to back, us, with 4 parts, with 16 and now (up to 512 tokens): 60
// sequences x 1024 columns 52, 28 and 28; 256 x 256 16.7, 17.5 and 14.9; up to 4
// tokens: 60 x 256 3.9, 4.7 and 4.0; 4096 x 1024 16.8, 35.7 and 17.8. The first
// 256 threads then compute the head logits with fixed-order reductions and thread
// 0 applies the softmax and writes the request's output row.
// POOL_COLS: columns of 16 parts summed at a time (32 KB of LDS).
constexpr int POOL_SHORT = 64, POOL_PARTS = 16, POOL_COLS = 512;

// A wave's parts of columns [0, n) of h: parts p0 .. p0 + PP - 1 of `parts`, U
// tokens of each at a time, to sums[p ld + c]. With PP > 1 or U > 4 every part
// has at least one token.
template <int PP, int U>
__device__ __forceinline__ void pool_sum(const float* __restrict__ h, int ldh, int n, bool vec, int L, int parts, int p0,
                                         float* sums, int ld, int lane) {
  int t0[PP], t1[PP];
#pragma unroll
  for (int i = 0; i < PP; ++i) {
    t0[i] = L * (p0 + i) / parts;
    t1[i] = L * (p0 + i + 1) / parts;
  }
  if (vec) {
    const int least = PP == 1 ? t1[0] - t0[0] : L / parts;  // tokens of a part: this many or one more
    for (int c = lane * 4; c < n; c += 256) {
      f32x4_t s[PP], v[PP][U];
#pragma unroll
      for (int i = 0; i < PP; ++i) s[i] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
      int k = 0;
      for (; k + U <= least; k += U) {
#pragma unroll
        for (int i = 0; i < PP; ++i)
#pragma unroll
          for (int u = 0; u < U; ++u) v[i][u] = *(const f32x4_t*)(h + (int64_t)(t0[i] + k + u) * ldh + c);
#pragma unroll
        for (int i = 0; i < PP; ++i)
#pragma unroll
          for (int u = 0; u < U; ++u) s[i] += v[i][u];
      }
      if constexpr (PP == 1 && U <= 4) {
        for (; k < least; ++k) s[0] += *(const f32x4_t*)(h + (int64_t)(t0[0] + k) * ldh + c);
      } else {  // at most U tokens of each part are left: loads past them repeat its last one
#pragma unroll
        for (int i = 0; i < PP; ++i)
#pragma unroll
          for (int u = 0; u < U; ++u) v[i][u] = *(const f32x4_t*)(h + (int64_t)min(t0[i] + k + u, t1[i] - 1) * ldh + c);
#pragma unroll
        for (int i = 0; i < PP; ++i)
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (t0[i] + k + u < t1[i]) s[i] += v[i][u];
      }
#pragma unroll
      for (int i = 0; i < PP; ++i) *(f32x4_t*)&sums[(p0 + i) * ld + c] = s[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < PP; ++i)
      for (int c = lane; c < n; c += 64) {
        float s = 0.f;
        for (int t = t0[i]; t < t1[i]; ++t) s += h[(int64_t)t * ldh + c];
        sums[(p0 + i) * ld + c] = s;
      }
  }
}

// LONG: slots of more than POOL_SHORT tokens.
template <int NW, bool LONG>
__global__ __launch_bounds__(NW * 64) void k_seqpool(const rb_k_row* __restrict__ rows, int n_seqs, int T,
                                                     int64_t packed_rows, const float* __restrict__ H, int ldh, int D,
                                                     const float* __restrict__ Wh,
                                                     const float* __restrict__ bh, int n_out, int act,
                                                     float* __restrict__ out) {
  const int r = blockIdx.x;
  const rb_k_row rw = rows[r];
  if (rw.out < 0) return;
  int L = (int)min(max(rw.aux, (int64_t)0), (int64_t)T);  // reads stay inside the slot
  // packed tokens: the sequence's rows [rows[r].lens, + L) of packed_rows
  if (packed_rows > 0 && (rw.lens < 0 || rw.lens + L > packed_rows)) L = 0;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  extern __shared__ float pool_lds[];  // the pooled row, then the partial sums of a pass of columns
  float* pooled = pool_lds;
  float* sums = pool_lds + (D + 3) / 4 * 4;
  __shared__ float part[4][POOL_MAX_OUT];
  const float* h = H + (packed_rows > 0 ? rw.lens : (int64_t)r * T) * ldh;
  const bool vec = (D & 3) == 0 && (ldh & 3) == 0;
  const float inv = 1.f / (float)max(L, 1);
  if (!LONG || L <= POOL_SHORT) {
    if (NW == 4 || wid < 4) pool_sum<1, 4>(h, ldh, D, vec, L, 4, wid, sums, D, lane);
    __syncthreads();
    for (int c = tid; c < D; c += NW * 64)
      pooled[c] = (((sums[c] + sums[D + c]) + sums[2 * D + c]) + sums[3 * D + c]) * inv;
    __syncthreads();
  } else {
    constexpr int PP = POOL_PARTS / NW;
    const int ld = min(D, POOL_COLS);
    for (int c0 = 0; c0 < D; c0 += POOL_COLS) {
      const int n = min(D - c0, POOL_COLS);
      pool_sum<PP, 8 / PP>(h + c0, ldh, n, vec, L, POOL_PARTS, wid * PP, sums, ld, lane);
      __syncthreads();
      for (int c = tid; c < n; c += NW * 64) {
        float s = 0.f;
#pragma unroll
        for (int p = 0; p < POOL_PARTS; ++p) s += sums[p * ld + c];
        pooled[c0 + c] = s * inv;
      }
      __syncthreads();
    }
  }
  for (int j = 0; j < n_out && tid < 256; ++j) {
    float s = 0.f;
    for (int c = tid; c < D; c += 256) s += Wh[(int64_t)j * D + c] * pooled[c];
    s = wave_sum(s);
    if (lane == 0) part[wid][j] = s;
  }
  __syncthreads();
  if (tid == 0) {
    float z[POOL_MAX_OUT];
    float mx = -INFINITY;
    for (int j = 0; j < n_out; ++j) {
      z[j] = ((part[0][j] + part[1][j]) + (part[2][j] + part[3][j])) + bh[j];
      mx = fmaxf(mx, z[j]);
    }
    if (act == RB_ACT_SOFTMAX) {
      float den = 0.f;
      for (int j = 0; j < n_out; ++j) {
        z[j] = expf(z[j] - mx);
        den += z[j];
      }
      for (int j = 0; j < n_out; ++j) out[rw.out + j] = z[j] / den;
    } else {
      for (int j = 0; j < n_out; ++j) out[rw.out + j] = z[j];
    }
  }
}

// Split: TPR threads per row, 256 / TPR rows per workgroup. With V = 4 a row
// whose output offset is a multiple of 4 floats is copied with 16-byte loads
// and stores (Y rows always are; output rows of a mixed-width arena may not
// be, and those take the scalar path).
template <int V>
__global__ __launch_bounds__(256) void k_split(const rb_k_row* __restrict__ rows, int n, int tpr,
                                               const float* __restrict__ Y, int ldy, int d_out,
                                               float* __restrict__ out) {
  const int rpb = 256 / tpr;
  const int r = blockIdx.x * rpb + threadIdx.x / tpr;
  if (r >= n) return;
  const int64_t o = rows[r].out;
  if (o < 0) return;
  const float* y = Y + (int64_t)r * ldy;
  const int t = threadIdx.x % tpr;
  if (V == 4 && (o & 3) == 0) {
    for (int c = t * 4; c < d_out; c += tpr * 4) *(float4*)(out + o + c) = *(const float4*)(y + c);
  } else {
    for (int c = t; c < d_out; c += tpr) out[o + c] = y[c];
  }
}

inline unsigned blocks_for(int64_t threads) { return (unsigned)((threads + 255) / 256); }

}  // namespace

// Runtime support (not part of the C ABI): the arena offset of every packed
// token row of a sequence group.
rb_status rb_token_rows(hipStream_t s, const rb_k_row* rows, int n_slots, int T, int64_t dense_len, int d_in,
                        int64_t* src, int64_t n_src, int* err) {
  if (n_slots < 1) return RB_OK;
  hipLaunchKernelGGL(k_token_rows, dim3((unsigned)((n_slots + 3) / 4)), dim3(256), 0, s, rows, n_slots, T, dense_len, d_in,
                     src, n_src, err);
  return launch_status();
}

// ---------------------------------------------------------------- static scratch

namespace {
// Work memory of the allocation-free launch-group entry point: one copy per
// GPU, resident from the code object's load until the process ends. Host code
// never passes this name to a kernel; it uses the device address looked up
// per device with hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[RB_STATIC_SCRATCH_BYTES];

constexpr int SCRATCH_MAX_DEVICES = 64;
std::mutex scratch_mu;
void* scratch_ptr[SCRATCH_MAX_DEVICES];
bool scratch_looked_up[SCRATCH_MAX_DEVICES];
}  // namespace

// Runtime support (not part of the C ABI): look up, once per device and with
// that device current, the device address of its copy of the scratch array.
rb_status rb_static_scratch_setup(int device) {
  if (device < 0 || device >= SCRATCH_MAX_DEVICES) return RB_EDEVICE;
  std::lock_guard<std::mutex> lk(scratch_mu);
  if (!scratch_looked_up[device]) {
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess) return RB_EDEVICE;
    if (cur != device && hipSetDevice(device) != hipSuccess) return RB_EDEVICE;
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess || !p) return RB_EDEVICE;
    scratch_ptr[device] = p;
    scratch_looked_up[device] = true;
  }
  return RB_OK;
}

// The device address of the device's scratch copy (nullptr before
// rb_static_scratch_setup succeeded on it).
void* rb_static_scratch(int device) {
  if (device < 0 || device >= SCRATCH_MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lk(scratch_mu);
  return scratch_looked_up[device] ? scratch_ptr[device] : nullptr;
}

// ---------------------------------------------------------------- cache scrub

namespace {
// Reads bytes of buf (a multiple of 16) so that L2 and the Infinity Cache hold
// only its clean lines afterwards; the loads feed a value stored only in a
// case that never happens, so they are not removed.
__global__ __launch_bounds__(256) void k_scrub(const u32x4_t* __restrict__ buf, int64_t n, unsigned* sink) {
  u32x4_t x = {0u, 0u, 0u, 0u};
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) x ^= buf[i];
  if (x.x == 0x9e3779b9u && x.y == 0x7f4a7c15u && x.z == 0xf39cc060u && x.w == 0x5cedc834u) sink[0] = 1u;
}
}  // namespace

// Cold-cache profiling support for the scheduler (not part of the C ABI).
void rb_scrub_caches(hipStream_t stream, const void* buf, size_t bytes, unsigned* sink) {
  hipLaunchKernelGGL(k_scrub, dim3(4096), dim3(256), 0, stream, (const u32x4_t*)buf, (int64_t)(bytes / 16), sink);
}

// ---------------------------------------------------------------- kernel ABI

extern "C" {

// rb_k_route (runtime support, not part of the C ABI): with `ends` also the end
// of every bag among its row's ids, table after table; with `fill` the rows that
// no batch covers become padding; max_rows: the most rows a batch has.
rb_status rb_route_bags(void* stream, int32_t kind, const rb_k_batch* batches, int32_t n_batches,
                        const rb_k_req* reqs, int32_t n_reqs, const int32_t* lens, int64_t lens_len, int32_t d_in,
                        int32_t d_out, int32_t n_tables, rb_k_row* rows, int32_t n_rows_total, int64_t out_len,
                        int32_t* ends, int32_t fill, int32_t max_rows, int32_t* err) {
  if (n_batches < 0 || n_reqs < 0 || n_rows_total < 0 || lens_len < 0 || out_len < 0 || !batches || !rows ||
      !err || d_in < 1 || d_out < 1)
    return RB_EINVAL;
  if (n_reqs > 0 && !reqs) return RB_EINVAL;
  if (kind < RB_MODEL_MLP || kind > RB_MODEL_SEQPOOL) return RB_EINVAL;
  if (kind != RB_MODEL_MLP && !lens) return RB_EINVAL;
  if (kind == RB_MODEL_RANKING && (n_tables < 1 || n_tables > MAX_TABLES)) return RB_EINVAL;
  if (n_batches == 0) return RB_OK;
  if (fill && n_batches > ROUTE_NT) {
    if (n_rows_total > 0)
      hipLaunchKernelGGL(k_fill_rows, dim3((unsigned)(((int64_t)n_rows_total + 255) / 256)), dim3(256), 0,
                         (hipStream_t)stream, rows, n_rows_total);
    fill = 0;
  }
#define RB_R(MAXR)                                                                                                    \
  hipLaunchKernelGGL(k_route<MAXR>, dim3(n_batches), dim3(ROUTE_NT), 0, (hipStream_t)stream, kind, batches, n_batches, \
                     reqs, n_reqs, lens, lens_len, d_in, d_out, n_tables, rows, n_rows_total, out_len, ends, fill, err)
  if (max_rows <= 512) RB_R(512);
  else RB_R(ROUTE_MAX_ROWS);
#undef RB_R
  return launch_status();
}

rb_status rb_k_route(void* stream, int32_t kind, const rb_k_batch* batches, int32_t n_batches,
                     const rb_k_req* reqs, int32_t n_reqs, const int32_t* lens, int64_t lens_len, int32_t d_in,
                     int32_t d_out, int32_t n_tables, rb_k_row* rows, int32_t n_rows_total, int64_t out_len,
                     int32_t* err) {
  return rb_route_bags(stream, kind, batches, n_batches, reqs, n_reqs, lens, lens_len, d_in, d_out, n_tables, rows,
                       n_rows_total, out_len, nullptr, 0, ROUTE_MAX_ROWS, err);
}

rb_status rb_k_assemble(void* stream, const rb_k_row* rows, int32_t n_rows_total, int32_t seq_T,
                        int32_t seq_real_only, const float* dense, int64_t dense_len, int32_t d_in, void* X,
                        int32_t ldx, int32_t out_bf16, float pad, int32_t* err) {
  if (n_rows_total < 0 || seq_T < 0 || d_in < 1 || ldx < d_in || (ldx & 7) || !rows || !X || !err)
    return RB_EINVAL;
  if (seq_real_only < 0 || seq_real_only > 2) return RB_EINVAL;
  if (seq_real_only && (seq_T == 0 || n_rows_total % seq_T || out_bf16)) return RB_EINVAL;
  if (n_rows_total == 0) return RB_OK;
  auto lg2 = [](int v) { int l = 0; while ((1 << l) < v) ++l; return (1 << l) == v ? l : -1; };
  if (seq_real_only) {
    const dim3 grid(n_rows_total / seq_T, (seq_T + SEQ_TOK - 1) / SEQ_TOK);
    if (seq_real_only == 2)
      hipLaunchKernelGGL(k_assemble_seq<true>, grid, dim3(256), 0, (hipStream_t)stream, rows, seq_T, dense, dense_len,
                         d_in, (float*)X, ldx, (int64_t)n_rows_total, err, lg2(ldx / 8));
    else
      hipLaunchKernelGGL(k_assemble_seq<false>, grid, dim3(256), 0, (hipStream_t)stream, rows, seq_T, dense,
                         dense_len, d_in, (float*)X, ldx, (int64_t)n_rows_total, err, lg2(ldx / 8));
    return launch_status();
  }
  const int64_t threads = (int64_t)n_rows_total * (ldx / 8);
  const unsigned g = blocks_for(threads);
  const int lg_c = lg2(ldx / 8), lg_t = seq_T > 0 ? lg2(seq_T) : 0;
  const bool pow2 = lg_c >= 0 && lg_t >= 0 && (int64_t)g * 256 < ((int64_t)1 << 31);
  hipStream_t hs = (hipStream_t)stream;
#define RB_ASM(B, P)                                                                                         \
  hipLaunchKernelGGL((k_assemble<B, P>), dim3(g), dim3(256), 0, hs, rows, n_rows_total, seq_T, dense, dense_len, \
                     d_in, X, ldx, pad, err, lg_c, lg_t)
  if (out_bf16) {
    if (pow2) RB_ASM(true, true);
    else RB_ASM(true, false);
  } else {
    if (pow2) RB_ASM(false, true);
    else RB_ASM(false, false);
  }
#undef RB_ASM
  return launch_status();
}

rb_status rb_k_embbag_dedup(void* stream, const rb_k_row* rows, int32_t n_rows_total, const int32_t* lens,
                            const int32_t* ids, int64_t ids_len, const void* const* tables, int32_t n_tables,
                            int64_t table_rows, int32_t emb_dim, const float* dense, int32_t n_dense, void* X,
                            int32_t ldx, float pad, int32_t* err) {
  if (emb_dim != EMB_DIM || n_tables < 1 || n_tables > MAX_TABLES || n_dense < 0 || n_dense > 256 ||
      table_rows < 1 || table_rows > INT32_MAX || ids_len < 0)
    return RB_EINVAL;
  if (n_rows_total < 0 || ldx < n_tables * EMB_DIM + n_dense || (ldx & 7) || !rows || !X || !err || !tables)
    return RB_EINVAL;
  if (n_rows_total == 0) return RB_OK;
  const unsigned grid = (unsigned)((n_rows_total + DD_ROWS - 1) / DD_ROWS) * n_tables;
  hipLaunchKernelGGL(k_embbag_dedup, dim3(grid), dim3(DD_NT), 0, (hipStream_t)stream, rows, n_rows_total, lens, ids,
                     ids_len, (const bf16_t* const*)tables, n_tables, table_rows, dense, n_dense, (bf16_t*)X, ldx,
                     pad, err);
  return launch_status();
}

// rb_k_embbag with the bags' ends from rb_route_bags (runtime support, not
// part of the C ABI; nullptr: from the lengths).
rb_status rb_embbag_ends(void* stream, const rb_k_row* rows, int32_t n_rows_total, const int32_t* lens,
                         const int32_t* ends, const int32_t* ids, int64_t ids_len, const void* const* tables,
                         int32_t n_tables, int64_t table_rows, int32_t emb_dim, const float* dense, int32_t n_dense,
                         void* X, int32_t ldx, float pad, int32_t* err) {
  if (emb_dim != EMB_DIM || n_tables < 1 || n_tables > MAX_TABLES || n_dense < 0 || n_dense > 256 ||
      table_rows < 1 || ids_len < 0)
    return RB_EINVAL;
  if (n_rows_total < 0 || ldx < n_tables * EMB_DIM + n_dense || (ldx & 7) || !rows || !X || !err || !tables)
    return RB_EINVAL;
  if (n_rows_total == 0) return RB_OK;
  // 32-bit byte offsets into the ids and into a table, with room for one that
  // is out of range
  const bool big = table_rows > 0xffffff00ll / (EMB_DIM * 2) || ids_len > 0xffffff00ll / 4;
  // bags per wave: 32 once that gives every compute unit 48 waves, 16 from 24
  // waves on, else 8 (26 bags a row: 32768 rows 105 us with 32, 110 with 16, 121
  // with 8; 4096 rows 24, 17 and 17; 64 rows 11, 8.7 and 5.7)
  const int64_t bags = (int64_t)n_rows_total * n_tables, cus = device_cus();
  // Without the ends 8: the lengths that a wave reads for each round's bags, one
  // round after another, cost more than the longer waves save (32768 rows: 189 us
  // with 32, 172 with 16, 154 with 8). Tables or ids past 32-bit offsets take the
  // same numbers (26 bags a row of a 4 GiB table: 512 rows 20.2
  // us with 32, 8.0 with 8; 4096 rows 38.3 and 30.5).
  const int rounds = !ends ? 1 : (bags >= 32 * 48 * cus ? 4 : (bags >= 16 * 24 * cus ? 2 : 1));
#define RB_E(R, B)                                                                                                   \
  hipLaunchKernelGGL((k_embbag<R, B>), dim3((unsigned)((n_rows_total + 32 * R - 1) / (32 * R)) * n_tables), dim3(256), 0, \
                     (hipStream_t)stream, rows, n_rows_total, lens, ends, ids, ids_len, (const bf16_t* const*)tables, \
                     n_tables, table_rows, dense, n_dense, (bf16_t*)X, ldx, pad, err)
  if (big) {
    if (rounds == 4) RB_E(4, true);
    else if (rounds == 2) RB_E(2, true);
    else RB_E(1, true);
  } else {
    if (rounds == 4) RB_E(4, false);
    else if (rounds == 2) RB_E(2, false);
    else RB_E(1, false);
  }
#undef RB_E
  return launch_status();
}

rb_status rb_k_embbag(void* stream, const rb_k_row* rows, int32_t n_rows_total, const int32_t* lens,
                      const int32_t* ids, int64_t ids_len, const void* const* tables, int32_t n_tables,
                      int64_t table_rows, int32_t emb_dim, const float* dense, int32_t n_dense, void* X, int32_t ldx,
                      float pad, int32_t* err) {
  return rb_embbag_ends(stream, rows, n_rows_total, lens, nullptr, ids, ids_len, tables, n_tables, table_rows, emb_dim,
                        dense, n_dense, X, ldx, pad, err);
}

rb_status rb_k_head(void* stream, const rb_k_row* rows, int32_t n_rows_total, const void* H, int32_t ldh,
                    const void* w, float b, int32_t K, int32_t act, float* out) {
  if (n_rows_total < 0 || K < 1 || ldh < K || !rows || !H || !w || !out) return RB_EINVAL;
  if (act != RB_ACT_NONE && act != RB_ACT_SIGMOID) return RB_EINVAL;
  if (n_rows_total == 0) return RB_OK;
  const unsigned g = (unsigned)((n_rows_total + 15) / 16);
  // 16-byte loads when every row and the weight vector start 16-byte aligned
  const int vec = (K % 8 == 0) && (ldh % 8 == 0) && ((uintptr_t)H % 16 == 0) && ((uintptr_t)w % 16 == 0);
  if (act == RB_ACT_SIGMOID)
    hipLaunchKernelGGL(k_head<RB_ACT_SIGMOID>, dim3(g), dim3(256), 0, (hipStream_t)stream, rows, n_rows_total,
                       (const bf16_t*)H, ldh, (const bf16_t*)w, b, K, vec, out);
  else
    hipLaunchKernelGGL(k_head<RB_ACT_NONE>, dim3(g), dim3(256), 0, (hipStream_t)stream, rows, n_rows_total,
                       (const bf16_t*)H, ldh, (const bf16_t*)w, b, K, vec, out);
  return launch_status();
}

rb_status rb_k_mlp_tail(void* stream, const rb_k_row* rows, int32_t n_rows_total, const void* H1, int32_t ldh1,
                        int32_t K2, const void* W2, int32_t ldw2, const float* b2, const void* W3, int32_t ldw3,
                        const float* b3, const void* w4, float b4, int32_t act, float* out) {
  if (n_rows_total < 0 || K2 < MT_KS || K2 % MT_KS || ldh1 < K2 || ldw2 < K2 || ldw3 < MT_N2) return RB_EINVAL;
  if ((ldh1 & 7) || (ldw2 & 7) || (ldw3 & 7) || !rows || !H1 || !W2 || !b2 || !W3 || !b3 || !w4 || !out)
    return RB_EINVAL;
  if (((uintptr_t)H1 & 15) || ((uintptr_t)W2 & 15) || ((uintptr_t)W3 & 15) || ((uintptr_t)w4 & 15)) return RB_EINVAL;
  if (act != RB_ACT_NONE && act != RB_ACT_SIGMOID) return RB_EINVAL;
  if (n_rows_total == 0) return RB_OK;
  const unsigned g = (unsigned)((n_rows_total + MT_BM - 1) / MT_BM);
  if (act == RB_ACT_SIGMOID)
    hipLaunchKernelGGL(k_mlp_tail<RB_ACT_SIGMOID>, dim3(g), dim3(MT_NT), 0, (hipStream_t)stream, (const bf16_t*)H1,
                       ldh1, K2, (const bf16_t*)W2, ldw2, b2, (const bf16_t*)W3, ldw3, b3, (const bf16_t*)w4, b4, rows,
                       n_rows_total, out);
  else
    hipLaunchKernelGGL(k_mlp_tail<RB_ACT_NONE>, dim3(g), dim3(MT_NT), 0, (hipStream_t)stream, (const bf16_t*)H1,
                       ldh1, K2, (const bf16_t*)W2, ldw2, b2, (const bf16_t*)W3, ldw3, b3, (const bf16_t*)w4, b4, rows,
                       n_rows_total, out);
  return launch_status();
}

rb_status rb_k_seqpool(void* stream, const rb_k_row* rows, int32_t n_seqs, int32_t seq_T, int64_t packed_rows,
                       const float* H, int32_t ldh, int32_t D, const float* Wh, const float* bh, int32_t n_out,
                       int32_t act, float* out) {
  if (n_seqs < 0 || seq_T < 1 || packed_rows < 0 || D < 1 || D > POOL_MAX_D || ldh < D || n_out < 1 ||
      n_out > POOL_MAX_OUT)
    return RB_EINVAL;
  if (act != RB_ACT_NONE && act != RB_ACT_SOFTMAX) return RB_EINVAL;
  if (!rows || !H || !Wh || !bh || !out) return RB_EINVAL;
  if (n_seqs == 0) return RB_OK;
  // the pooled row (whole 16 bytes) and the partial sums of 4 parts or, for long slots, of a pass of 16
  const size_t sums = seq_T <= POOL_SHORT ? 4 * D : std::max(4 * D, POOL_PARTS * std::min(D, POOL_COLS));
  const size_t lds = ((size_t)(D + 3) / 4 * 4 + sums) * sizeof(float);
#define RB_P(NW, LONG)                                                                                               \
  hipLaunchKernelGGL((k_seqpool<NW, LONG>), dim3(n_seqs), dim3(NW * 64), lds, (hipStream_t)stream, rows, n_seqs, seq_T, \
                     packed_rows, H, ldh, D, Wh, bh, n_out, act, out)
  if (seq_T <= POOL_SHORT) RB_P(4, false);
  else if (n_seqs < (int)device_cus()) RB_P(16, true);  // a launch takes as long as one workgroup
  else RB_P(4, true);
#undef RB_P
  return launch_status();
}

rb_status rb_k_split(void* stream, const rb_k_row* rows, int32_t n_rows_total, const float* Y, int32_t ldy,
                     int32_t d_out, float* out) {
  if (n_rows_total < 0 || d_out < 1 || ldy < d_out || !rows || !Y || !out) return RB_EINVAL;
  if (n_rows_total == 0) return RB_OK;
  // 16-byte path: width, row stride and both bases multiples of 4 floats
  const bool v4 = (d_out % 4) == 0 && (ldy % 4) == 0 && ((uintptr_t)Y % 16) == 0 && ((uintptr_t)out % 16) == 0;
  const int per = v4 ? d_out / 4 : d_out;
  int tpr = 1;
  while (tpr < per && tpr < 256) tpr <<= 1;
  const unsigned g = (unsigned)((n_rows_total + 256 / tpr - 1) / (256 / tpr));
  if (v4)
    hipLaunchKernelGGL(k_split<4>, dim3(g), dim3(256), 0, (hipStream_t)stream, rows, n_rows_total, tpr, Y, ldy,
                       d_out, out);
  else
    hipLaunchKernelGGL(k_split<1>, dim3(g), dim3(256), 0, (hipStream_t)stream, rows, n_rows_total, tpr, Y, ldy,
                       d_out, out);
  return launch_status();
}

}  // extern "C"
