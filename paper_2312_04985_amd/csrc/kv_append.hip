// Cache maintenance: append key/value rows, keep the S-contiguous key copy and the running
// mean value vector in step (Section 3 "Mean value reallocation"; Appendix F "Storing K twice").
#include "append_plan.h"
#include "decode_stages.h"

namespace sparq {

namespace {

// ---- one row per sequence: the per-token path of the decode loop ----
// One workgroup per sequence so that seq_lens[b] is read by everyone before it is bumped.
// A thread moves one 16-byte chunk (8 channels) of one KV head at a time.
template <class T>
__global__ __launch_bounds__(512) void append_one_row(const AppendArgs a) {
  const int b = blockIdx.x, tid = threadIdx.x;
  const int S = a.seq_lens[b];
  int n = a.n_new_per_seq ? a.n_new_per_seq[b] : 1;
  n = n < 0 ? 0 : (n > 1 ? 1 : n);
  const bool in_place = a.v_mean_out == a.v_mean;
  const bool full = S < 0 || S + 1 > a.S_max;
  if (n == 0 || full) {      // nothing appended: the state is carried over unchanged
    if (full && n != 0 && tid == 0) atomicOr(a.err, 1);
    if (!in_place) {
      for (int i = tid; i < a.H_kv * a.d_h; i += 512) {
        const size_t e = (size_t)b * a.H_kv * a.d_h + i;
        a.v_mean_out[e] = a.v_mean[e];
      }
      if (tid == 0) a.seq_lens_out[b] = S;
    }
    return;
  }
  const int cpr = a.d_h / 8;                  // 16-byte chunks per row
  const int n_chunks = a.H_kv * cpr;
  const float inv = 1.0f / (float)(S + 1);
  for (int c = tid; c < n_chunks; c += 512) {
    const int hk = c / cpr, j0 = (c - hk * cpr) * 8;
    const size_t head = (size_t)b * a.H_kv + hk;
    const uint4 kc = load16(reinterpret_cast<const uint16_t*>(a.k_new) + head * a.d_h + j0);
    const uint4 vc = load16(reinterpret_cast<const uint16_t*>(a.v_new) + head * a.d_h + j0);
    uint16_t* Krow = reinterpret_cast<uint16_t*>(a.K) + (head * a.S_stride + S) * a.d_h + j0;
    uint16_t* Vrow = reinterpret_cast<uint16_t*>(a.V) + (head * a.S_stride + S) * a.d_h + j0;
    *reinterpret_cast<uint4*>(Krow) = kc;
    *reinterpret_cast<uint4*>(Vrow) = vc;
    // the same 8 key elements go down column S of the S-contiguous copy (2-byte stores)
    // the S-contiguous copy advances 8 positions at a time: when this row completes a group of 8, the
    // thread writes columns S-7 .. S of its 8 channels (rows S-7 .. S-1 come back from K)
    if (a.Kt && ((S + 1) & 7) == 0) {   // null: the cache keeps K once
      const uint32_t kw[4] = {kc.x, kc.y, kc.z, kc.w};
#pragma unroll
      for (int e = 0; e < 8; ++e)
        flush_key_columns(reinterpret_cast<uint16_t*>(a.Kt) + head * a.d_h * (size_t)a.S_stride,
                          reinterpret_cast<const uint16_t*>(a.K) + head * a.S_stride * (size_t)a.d_h, a.S_stride, a.d_h, S + 1,
                          j0 + e, (uint16_t)((e & 1) ? (kw[e >> 1] >> 16) : (kw[e >> 1] & 0xffffu)));
    }
    // running mean: v_mean += (v - v_mean) / (S + 1)
    const float* vm = a.v_mean + head * a.d_h + j0;
    float* vo = a.v_mean_out + head * a.d_h + j0;
    float4 m0 = *reinterpret_cast<const float4*>(vm), m1 = *reinterpret_cast<const float4*>(vm + 4);
    if (S == 0) m0 = m1 = make_float4(0.f, 0.f, 0.f, 0.f);   // the mean of no rows: whatever the buffer held is ignored
    float f[8];
    unpack8<T>(vc, f);
    m0.x += (f[0] - m0.x) * inv; m0.y += (f[1] - m0.y) * inv; m0.z += (f[2] - m0.z) * inv; m0.w += (f[3] - m0.w) * inv;
    m1.x += (f[4] - m1.x) * inv; m1.y += (f[5] - m1.y) * inv; m1.z += (f[6] - m1.z) * inv; m1.w += (f[7] - m1.w) * inv;
    *reinterpret_cast<float4*>(vo) = m0;
    *reinterpret_cast<float4*>(vo + 4) = m1;
  }
  __syncthreads();
  if (tid == 0) a.seq_lens_out[b] = S + 1;
}

// ---- many rows per sequence (prefill / cache construction) ----
// The rows of a (sequence, KV head) are cut into tiles of ATP positions, aligned to 64 positions of the cache so that a
// tile's columns of Kt are whole 128-byte lines, and dealt to n_split workgroups: a prompt for one sequence with 8 KV
// heads is 8 x 249 tiles.  A thread owns 8 channels of 8 consecutive positions: it copies its 8 pieces of K and of V,
// transposes the keys in registers and hands them over through LDS as 16-byte pieces of a channel row, which leave as
// runs of 2 ATP bytes.  Bound by HBM (2 rows in, 3 out); value columns are summed in fp64, one partial sum per
// workgroup.  With few workgroups the last one of a KV head folds them into the mean, and the last KV head of a sequence
// advances its length (counters in the control block); with many, whose stores saturate the memory that every such
// hand-over waits for, a second launch does it, append_finish or bump_seq_lens (see launch_rows_dh).
// Measured (whole call; before: one workgroup per KV head, columns in 2-byte stores): a prompt of 31 777 rows for 8 KV
// heads, d_h 128 (325 MB read and written) 2301 -> 70 us; chunks of 1-512 rows for 512 KV heads (169 MB) 63 -> 42 us.  (With a
// branch around each row's loads the compiler put each one's wait behind it: 79 and 48 us.)
constexpr int BT = kAppendThreads;
// (rows of K and V leave as non-temporal stores: 84 -> 78 us for that prompt; the columns of Kt do not: 78 -> 82)
__device__ __forceinline__ void store16_nt(void* p, const uint4& c) {
  u32x4 v; v.x = c.x; v.y = c.y; v.z = c.z; v.w = c.w;
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
}
template <int DH>
constexpr int ATP = append_tile(DH);       // positions per tile

// the codes of positions 0 .. left - 1 of a group of 8, 16 bytes where it is whole
__device__ __forceinline__ void store_columns(uint16_t* dst, uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3, int left) {
  if (left >= 8) {
    *reinterpret_cast<uint4*>(dst) = make_uint4(x0, x1, x2, x3);
  } else {                               // the last, unfinished group: its positions only, as 4 + 2 + 1
    const uint64_t lo = x0 | ((uint64_t)x1 << 32), hi = x2 | ((uint64_t)x3 << 32);
    if (left & 4) *reinterpret_cast<uint64_t*>(dst) = lo;
    const uint64_t rest = left & 4 ? hi : lo;
    if (left & 2) *reinterpret_cast<uint32_t*>(dst + (left & 4)) = (uint32_t)rest;
    if (left & 1) dst[left & 6] = (uint16_t)(rest >> (left & 2 ? 32 : 0));
  }
}

template <class T, int DH>
__global__ __launch_bounds__(BT) void append_rows(const AppendArgs a) {
  constexpr int CPR = DH / 8;            // 16-byte pieces per row
  constexpr int RPP = BT / CPR;          // groups of 8 positions per tile
  constexpr int TP = ATP<DH>;
  __shared__ __align__(16) uint4 tile[DH * RPP];   // [channel][group ^ (channel / 8)]: no bank conflicts either way
  double (*colsum)[DH] = reinterpret_cast<double (*)[DH]>(tile);   // [RPP][DH], after the last tile
  __shared__ int last;
  const int tid = threadIdx.x;
  // Workgroups are dealt round-robin to the 8 XCDs: the head varies fastest, so that the workgroups that find no rows do not
  // all fall to the same ones (1024 KV heads x 200 rows, every second workgroup without rows: 77 -> 61 us).
  const int heads = a.B * a.H_kv, split = blockIdx.x / heads;
  const size_t head = blockIdx.x - split * heads;
  const int b = (int)(head / a.H_kv);
  const int S = a.seq_lens[b];
  int n = a.n_new_per_seq ? a.n_new_per_seq[b] : a.n_new;
  n = n < 0 ? 0 : (n > a.n_new ? a.n_new : n);
  const bool full = S < 0 || S + n > a.S_max;
  if (!a.tickets && a.n_split > 1 && split == 0 && tid == 0) a.span_ws[head] = make_int2(S, full ? 0 : n);
  if (n == 0) return;
  if (full) {
    if (split == 0 && tid == 0) atomicOr(a.err, 1);
    return;
  }
  const int sub = tid % CPR, grp = tid / CPR;
  const uint16_t* ksrc = reinterpret_cast<const uint16_t*>(a.k_new) + head * a.n_new * DH + sub * 8;   // row i is position S + i
  const uint16_t* vsrc = reinterpret_cast<const uint16_t*>(a.v_new) + head * a.n_new * DH + sub * 8;
  uint16_t* Khead = reinterpret_cast<uint16_t*>(a.K) + head * a.S_stride * (size_t)DH + sub * 8;
  uint16_t* Vhead = reinterpret_cast<uint16_t*>(a.V) + head * a.S_stride * (size_t)DH + sub * 8;
  uint16_t* Kthead = reinterpret_cast<uint16_t*>(a.Kt) + head * DH * (size_t)a.S_stride;
  const int E = S + n, S_fl = S & ~7;
  const AppendSplit plan{a.n_split, a.tiles_per_split};
  const AppendRun run = append_run(S, n, split, plan, DH);
  const int p_begin = run.begin, p_end = run.end;
  double sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int p0 = p_begin; p0 < p_end; p0 += TP) {
    const int p = p0 + grp * 8;          // this thread's 8 positions
    if (p + 8 > S_fl && p < p_end) {     // some of them belong to this call, or wait for their place in Kt
      // all 16 pieces are requested before the first is used: no branch around a load, the rows next to those of the call stand in
      uint4 kr[8], vr[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int q = p + e, i = q < S ? 0 : (q < E ? q - S : n - 1);
        // (S_fl <= q < S: cached before this call and not yet in the S-contiguous copy)
        kr[e] = load16(q < S ? Khead + (size_t)q * DH : ksrc + (size_t)i * DH);
        vr[e] = load16(vsrc + (size_t)i * DH);
      }
      if (a.Kt) {                        // null: the cache keeps K once
        uint4 w[8];
        transpose_piece(kr, w);
#pragma unroll
        for (int c = 0; c < 8; ++c) tile[(sub * 8 + c) * RPP + (grp ^ (sub & (RPP - 1)))] = w[c];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int q = p + e;
        if (q >= S && q < E) {
          store16_nt(Khead + (size_t)q * DH, kr[e]);
          store16_nt(Vhead + (size_t)q * DH, vr[e]);
          float f[8];
          unpack8<T>(vr[e], f);
#pragma unroll
          for (int c = 0; c < 8; ++c) sum[c] += (double)f[c];
        }
      }
    }
    if (a.Kt) {
      __syncthreads();
      // the groups that hold positions of this call, dealt evenly to the threads (a short append fills a few of RPP)
      const int u0 = p0 < S_fl ? (S_fl - p0) >> 3 : 0, u1 = (p_end - p0 + 7) >> 3, live = (u1 < RPP ? u1 : RPP) - u0;
      const float per_live = 1.0f / (float)live;
      for (int i = tid; i < DH * live; i += BT) {
        const int j = (int)(((float)i + 0.5f) * per_live), u = u0 + i - j * live, q = p0 + u * 8;   // i / live: i < 2^12
        const uint4 v = tile[j * RPP + (u ^ ((j >> 3) & (RPP - 1)))];
        uint16_t* dst = Kthead + (size_t)j * a.S_stride + q;
        store_columns(dst, v.x, v.y, v.z, v.w, E - q);
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) colsum[grp][sub * 8 + c] = sum[c];
  __syncthreads();
  if (tid < DH) {
    double tot = 0.0;
    for (int g = 0; g < RPP; ++g) tot += colsum[g][tid];
    if (a.n_split > 1) {                   // (only the partial sums of workgroups with rows are read)
      double* mine = a.part_ws + (head * a.n_split + split) * DH + tid;
      if (a.tickets) store_agent(mine, tot); else *mine = tot;
    } else {
      float* vm = a.v_mean + head * DH + tid;
      const double before = S > 0 ? (double)S * (double)*vm : 0.0;   // S = 0: whatever the buffer held is ignored
      *vm = (float)((before + tot) / (double)(S + n));
    }
  }
  if (!a.tickets) return;
  if (a.n_split > 1) {
    if (!last_to_arrive(a.tickets + a.B + head, append_arrivals(plan), &last)) return;
    // the partial sums dealt to BT / DH groups of threads, 16 in flight each (8 in flight for a channel's one thread: a whole
    // call of 32 768 rows for one KV head 25.3 us, so 22.9)
    constexpr int NG = BT / DH, FLY = 16;
    const int used = run.used, c = tid % DH, g = tid / DH;
    const double* part = a.part_ws + head * a.n_split * DH + c;
    double tot = 0.0;
    for (int s0 = g; s0 < used; s0 += NG * FLY) {
      double v[FLY];
#pragma unroll
      for (int t = 0; t < FLY; ++t) v[t] = load_agent(part + (size_t)(s0 + t * NG < used ? s0 + t * NG : used - 1) * DH);
#pragma unroll
      for (int t = 0; t < FLY; ++t) tot += s0 + t * NG < used ? v[t] : 0.0;
    }
    if (NG > 1) {
      colsum[g][c] = tot;
      __syncthreads();
    }
    if (g == 0) {
      float* vm = a.v_mean + head * DH + c;
      const double before = S > 0 ? (double)S * (double)*vm : 0.0;
#pragma unroll
      for (int o = 1; o < NG; ++o) tot += colsum[o][c];
      *vm = (float)((before + tot) / (double)(S + n));
    }
  }
  // Every workgroup of the sequence, those without rows among them, has read its length by the time its KV head is
  // counted: one that started after the length was written would take the new length for the old one.
  if (last_to_arrive(a.tickets + b, a.H_kv, &last) && tid == 0) a.seq_lens[b] = E;
}

// Up to kAppendShort rows for many KV heads: one workgroup per KV head, a thread moves 16-byte pieces of single rows, and
// the keys are transposed through LDS, 16 bytes of a channel row at a time.  Bound by round trips at few rows, by HBM and the
// lines of Kt that are written in part at many.  Measured (device us, against append_rows as it was): 512 heads of 128
// x 8 rows 14.0 -> 8.1, 2048 x 8 34.7 -> 17.3, 2048 x 64 56.5 -> 45.2.
template <class T, int DH>
__global__ __launch_bounds__(BT) void append_rows_short(const AppendArgs a) {
  constexpr int CPR = DH / 8, RPP = BT / CPR;
  constexpr int LD = DH + 2;                               // padded row: the groups' reads below fall into different banks
  constexpr int ROWS = (kAppendShort + 7 + 7) & ~7;
  __shared__ __align__(16) uint16_t tile[ROWS * LD];       // rows S_fl .. S + n - 1, row-major
  __shared__ double colsum[RPP][DH];
  const int tid = threadIdx.x;
  const size_t head = blockIdx.x;
  const int b = (int)(head / a.H_kv);
  const int S = a.seq_lens[b];
  int n = a.n_new_per_seq ? a.n_new_per_seq[b] : a.n_new;
  n = n < 0 ? 0 : (n > a.n_new ? a.n_new : n);
  if (n == 0) return;
  if (S < 0 || S + n > a.S_max) {
    if (tid == 0) atomicOr(a.err, 1);
    return;
  }
  float* vm = a.v_mean + head * DH + tid % DH;
  const float mean = *vm;                  // requested early, by all threads: no branch that waits for it
  const int sub = tid % CPR, row = tid / CPR;
  const uint16_t* ksrc = reinterpret_cast<const uint16_t*>(a.k_new) + head * a.n_new * DH + sub * 8;
  const uint16_t* vsrc = reinterpret_cast<const uint16_t*>(a.v_new) + head * a.n_new * DH + sub * 8;
  uint16_t* Khead = reinterpret_cast<uint16_t*>(a.K) + head * a.S_stride * (size_t)DH + sub * 8;
  uint16_t* Vhead = reinterpret_cast<uint16_t*>(a.V) + head * a.S_stride * (size_t)DH + sub * 8;
  const int E = S + n, S_fl = a.Kt ? S & ~7 : S;           // (rows S_fl .. S - 1 are cached and not yet in the S-contiguous copy)
  double sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int q = S_fl + row; q < E; q += RPP) {
    const int i = q < S ? 0 : q - S;
    const uint4 kc = load16(q < S ? Khead + (size_t)q * DH : ksrc + (size_t)i * DH);
    const uint4 vc = load16(vsrc + (size_t)i * DH);
    if (q >= S) {
      *reinterpret_cast<uint4*>(Khead + (size_t)q * DH) = kc;
      *reinterpret_cast<uint4*>(Vhead + (size_t)q * DH) = vc;
      float f[8];
      unpack8<T>(vc, f);
#pragma unroll
      for (int c = 0; c < 8; ++c) sum[c] += (double)f[c];
    }
    // (after the branch: in front of it, the piece of K would be waited for before that of V is asked for: 14.2 -> 16.4 us)
    uint32_t* dst = reinterpret_cast<uint32_t*>(tile + (q - S_fl) * LD + sub * 8);   // LD even: 4-byte aligned
    dst[0] = kc.x; dst[1] = kc.y; dst[2] = kc.z; dst[3] = kc.w;
  }
  __syncthreads();
  if (a.Kt) {
    uint16_t* Kthead = reinterpret_cast<uint16_t*>(a.Kt) + head * DH * (size_t)a.S_stride + S_fl;
    const int rows = E - S_fl, live = (rows + 7) >> 3;
    const float per_live = 1.0f / (float)live;
    for (int i = tid; i < DH * live; i += BT) {
      const int j = (int)(((float)i + 0.5f) * per_live), r = (i - j * live) * 8;      // i / live: i < 2^12
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 8; e += 2) w[e >> 1] = tile[(r + e) * LD + j] | ((uint32_t)tile[(r + e + 1) * LD + j] << 16);
      store_columns(Kthead + (size_t)j * a.S_stride + r, w[0], w[1], w[2], w[3], rows - r);
    }
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) colsum[row][sub * 8 + c] = sum[c];
  __syncthreads();
  if (tid < DH) {
    double tot = 0.0;
    for (int g = 0; g < RPP; ++g) tot += colsum[g][tid];
    const double before = S > 0 ? (double)S * (double)mean : 0.0;    // S = 0: whatever the buffer held is ignored
    *vm = (float)((before + tot) / (double)(S + n));
  }
}

// The means and lengths after append_rows over several workgroups per KV head: one workgroup per (sequence, KV head).
// The old length and the row count come from the workspace: seq_lens is written here.
// Bound by memory latency: the lengths, the old mean and the partial sums are requested together, the partial sums of
// workgroups that had no rows among them (never written, and left out).  THREADS = 1024 where a KV head has more than 16
// partial sums: THREADS / DH groups of 16 are in flight at once, which is all of them (128 at most) for d_h 64 and 128; at d_h 256
// it is 64, and heads with more take a second round.  (With 8 per thread in flight behind the lengths, a whole call: 31 777 rows
// for 8 KV heads 70.4 us, so 67.4.)
template <int DH, int THREADS>
__global__ __launch_bounds__(THREADS) void append_finish(const AppendArgs a) {
  constexpr int NG = THREADS / DH, FLY = 16;
  __shared__ double sm[NG][DH];
  const int c = threadIdx.x % DH, grp = threadIdx.x / DH;
  const size_t head = blockIdx.x;
  const int b = (int)(head / a.H_kv);
  const int2 sn = a.span_ws[head];
  float* vm = a.v_mean + head * DH + c;
  const float old = *vm;
  const double* part = a.part_ws + head * a.n_split * DH + c;
  double v[FLY];
  auto fetch = [&](int s0) {
#pragma unroll
    for (int t = 0; t < FLY; ++t) v[t] = s0 + t * NG < a.n_split ? part[(size_t)(s0 + t * NG) * DH] : 0.0;
  };
  fetch(grp);
  const int S = sn.x, n = sn.y;
  if (n == 0) return;
  const double before = S > 0 ? (double)S * (double)old : 0.0;     // S = 0: whatever the buffer held is ignored
  const int used = append_run(S, n, 0, AppendSplit{a.n_split, a.tiles_per_split}, DH).used;   // workgroups that had rows
  double tot = 0.0;
  for (int s0 = grp;;) {
#pragma unroll
    for (int t = 0; t < FLY; ++t) tot += s0 + t * NG < used ? v[t] : 0.0;
    s0 += NG * FLY;
    if (s0 >= used) break;
    fetch(s0);
  }
  sm[grp][c] = tot;
  __syncthreads();
  if (grp == 0) {
#pragma unroll
    for (int g = 1; g < NG; ++g) tot += sm[g][c];
    *vm = (float)((before + tot) / (double)(S + n));
  }
  if (head % a.H_kv == 0 && threadIdx.x == 0) a.seq_lens[b] = S + n;
}

// ---- the tiled single-copy key layout: tiles of 8 positions, channel-major inside a tile ----
// K element (position p, channel j) of a KV head lies at ((p / 8) d_h + j) 8 + p % 8; the rows of the
// positions 8 floor(S / 8) .. S - 1, which do not fill a tile yet, wait in a buffer of 8 rows per KV head
// (AppendArgs::Kt) and move into their tile, as one contiguous block, when the eighth arrives.

// the transposed piece of 8 rows x 8 channels as 128 contiguous bytes at `dst`
__device__ __forceinline__ void store_tile_piece(uint16_t* dst, const uint4 (&rows)[8]) {
  uint4 w[8];
  transpose_piece(rows, w);
#pragma unroll
  for (int c = 0; c < 8; ++c) reinterpret_cast<uint4*>(dst)[c] = w[c];
}

// one row per sequence: one workgroup per sequence, a thread moves one 16-byte chunk (8 channels) of one KV head
template <class T>
__global__ __launch_bounds__(512) void append_one_row_tiled(const AppendArgs a) {
  const int b = blockIdx.x, tid = threadIdx.x;
  const int S = a.seq_lens[b];
  int n = a.n_new_per_seq ? a.n_new_per_seq[b] : 1;
  n = n < 0 ? 0 : (n > 1 ? 1 : n);
  const bool in_place = a.v_mean_out == a.v_mean;
  const bool full = S < 0 || S + 1 > a.S_max;
  if (n == 0 || full) {      // nothing appended: the state is carried over unchanged
    if (full && n != 0 && tid == 0) atomicOr(a.err, 1);
    if (!in_place) {
      for (int i = tid; i < a.H_kv * a.d_h; i += 512) {
        const size_t e = (size_t)b * a.H_kv * a.d_h + i;
        a.v_mean_out[e] = a.v_mean[e];
      }
      if (tid == 0) a.seq_lens_out[b] = S;
    }
    return;
  }
  const int cpr = a.d_h / 8;
  const int n_chunks = a.H_kv * cpr;
  const float inv = 1.0f / (float)(S + 1);
  const int slot = S & 7;
  for (int c = tid; c < n_chunks; c += 512) {
    const int hk = c / cpr, j0 = (c - hk * cpr) * 8;
    const size_t head = (size_t)b * a.H_kv + hk;
    const uint4 kc = load16(reinterpret_cast<const uint16_t*>(a.k_new) + head * a.d_h + j0);
    const uint4 vc = load16(reinterpret_cast<const uint16_t*>(a.v_new) + head * a.d_h + j0);
    uint16_t* stage = reinterpret_cast<uint16_t*>(a.Kt) + head * (size_t)(8 * a.d_h);
    *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(a.V) + (head * a.S_stride + S) * a.d_h + j0) = vc;
    if (slot != 7) {
      *reinterpret_cast<uint4*>(stage + slot * a.d_h + j0) = kc;
    } else {               // the eighth row: this thread's 8 channels of the finished tile
      uint4 rows[8];
#pragma unroll
      for (int e = 0; e < 7; ++e) rows[e] = load16(stage + e * a.d_h + j0);
      rows[7] = kc;
      store_tile_piece(reinterpret_cast<uint16_t*>(a.K) + (head * a.S_stride + (size_t)(S - 7)) * a.d_h + (size_t)j0 * 8, rows);
    }
    const float* vm = a.v_mean + head * a.d_h + j0;
    float* vo = a.v_mean_out + head * a.d_h + j0;
    float4 m0 = *reinterpret_cast<const float4*>(vm), m1 = *reinterpret_cast<const float4*>(vm + 4);
    if (S == 0) m0 = m1 = make_float4(0.f, 0.f, 0.f, 0.f);
    float f[8];
    unpack8<T>(vc, f);
    m0.x += (f[0] - m0.x) * inv; m0.y += (f[1] - m0.y) * inv; m0.z += (f[2] - m0.z) * inv; m0.w += (f[3] - m0.w) * inv;
    m1.x += (f[4] - m1.x) * inv; m1.y += (f[5] - m1.y) * inv; m1.z += (f[6] - m1.z) * inv; m1.w += (f[7] - m1.w) * inv;
    *reinterpret_cast<float4*>(vo) = m0;
    *reinterpret_cast<float4*>(vo + 4) = m1;
  }
  __syncthreads();
  if (tid == 0) a.seq_lens_out[b] = S + 1;
}

// many rows per sequence: one workgroup per (sequence, KV head); the positions go tile by tile: thread (row e,
// chunk sub) of a tile brings its 16 bytes (from the buffer of waiting rows for positions cached before this
// call, else from k_new) into LDS, and the threads of the first row write the tile's 128-byte pieces; the rows
// of an unfinished last tile go (back) into the buffer.  V rows and the mean as in append_rows.
template <class T, int DH>
__global__ __launch_bounds__(BT) void append_rows_tiled(const AppendArgs a) {
  constexpr int CPR = DH / 8;            // 16-byte chunks per row
  constexpr int TPP = BT / (8 * CPR);    // tiles per pass (BT = 256: 4, 2 or 1)
  constexpr int RPP = BT / CPR;          // value rows per pass
  __shared__ __align__(16) uint16_t tile[TPP * 8 * DH];
  __shared__ double colsum[RPP][DH];
  const int tid = threadIdx.x;
  const size_t head = blockIdx.x;
  const int b = (int)(head / a.H_kv);
  const int S = a.seq_lens[b];
  int n = a.n_new_per_seq ? a.n_new_per_seq[b] : a.n_new;
  n = n < 0 ? 0 : (n > a.n_new ? a.n_new : n);
  if (n == 0) return;
  if (S < 0 || S + n > a.S_max) {
    if (tid == 0) atomicOr(a.err, 1);
    return;
  }
  const uint16_t* ksrc = reinterpret_cast<const uint16_t*>(a.k_new) + head * a.n_new * DH;
  const uint16_t* vsrc = reinterpret_cast<const uint16_t*>(a.v_new) + head * a.n_new * DH;
  uint16_t* Kdst = reinterpret_cast<uint16_t*>(a.K) + head * a.S_stride * (size_t)DH;
  uint16_t* stage = reinterpret_cast<uint16_t*>(a.Kt) + head * (size_t)(8 * DH);
  uint16_t* Vdst = reinterpret_cast<uint16_t*>(a.V) + (head * a.S_stride + S) * DH;
  // keys, tile by tile
  const int sub = tid % CPR, e = (tid / CPR) & 7, tl = tid / (8 * CPR);
  const int g_first = S >> 3, g_last = (S + n - 1) >> 3;
  for (int g0 = g_first; g0 <= g_last; g0 += TPP) {
    const int g = g0 + tl, p = g * 8 + e;                 // this thread's tile and position
    const bool have = g <= g_last && p < S + n;
    uint4 kc = make_uint4(0u, 0u, 0u, 0u);
    if (have) kc = p < S ? load16(stage + e * DH + sub * 8) : load16(ksrc + (size_t)(p - S) * DH + sub * 8);
    *reinterpret_cast<uint4*>(tile + (tl * 8 + e) * DH + sub * 8) = kc;
    __syncthreads();
    if (g <= g_last) {
      if (g * 8 + 8 <= S + n) {                           // a finished tile
        if (e == 0) {
          uint4 rows[8];
#pragma unroll
          for (int r = 0; r < 8; ++r) rows[r] = *reinterpret_cast<const uint4*>(tile + (tl * 8 + r) * DH + sub * 8);
          store_tile_piece(Kdst + ((size_t)g * DH + sub * 8) * 8, rows);
        }
      } else if (have && p >= S) {                        // a new row that waits for its tile
        *reinterpret_cast<uint4*>(stage + e * DH + sub * 8) = kc;
      }
    }
    __syncthreads();
  }
  // values and their column sums
  const int prow = tid / CPR;
  double sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int rr = prow; rr < n; rr += RPP) {
    const size_t off = (size_t)rr * DH + sub * 8;
    const uint4 vc = load16(vsrc + off);
    *reinterpret_cast<uint4*>(Vdst + off) = vc;
    float f[8];
    unpack8<T>(vc, f);
#pragma unroll
    for (int c = 0; c < 8; ++c) sum[c] += (double)f[c];
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) colsum[prow][sub * 8 + c] = sum[c];
  __syncthreads();
  if (tid < DH) {
    double tot = 0.0;
    for (int p = 0; p < RPP; ++p) tot += colsum[p][tid];
    float* vm = a.v_mean + head * DH + tid;
    const double before = S > 0 ? (double)S * (double)*vm : 0.0;
    *vm = (float)((before + tot) / (double)(S + n));
  }
}

__global__ void bump_seq_lens(const AppendArgs a) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= a.B) return;
  const int S = a.seq_lens[b];
  int n = a.n_new_per_seq ? a.n_new_per_seq[b] : a.n_new;
  n = n < 0 ? 0 : (n > a.n_new ? a.n_new : n);
  if (S >= 0 && S + n <= a.S_max) a.seq_lens[b] = S + n;
}

// Both probes: every workgroup streams one contiguous slab of the buffer (a grid-strided walk, where the 8
// loads of a thread are megabytes apart, reaches only ~5.0 TB/s here; contiguous slabs reach 6.2-6.4), 8
// independent 16-byte accesses per thread in flight, the read probe two batches deep.
__device__ __forceinline__ void probe_slab(size_t n16, size_t& begin, size_t& end) {
  const size_t chunk = (size_t)blockDim.x * 8;
  size_t per = (n16 + gridDim.x - 1) / gridDim.x;
  per = (per + chunk - 1) / chunk * chunk;
  begin = (size_t)blockIdx.x * per;
  end = begin + per < n16 ? begin + per : n16;
  if (begin > n16) begin = n16;
}

__global__ __launch_bounds__(256) void copy_probe(uint4* dst, const uint4* src, size_t n16) {
  size_t begin, end;
  probe_slab(n16, begin, end);
  const size_t T = blockDim.x;
  size_t i = begin + threadIdx.x;
  for (; i + 7 * T < end; i += 8 * T) {
    uint4 v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = load16(src + i + t * T);
#pragma unroll
    for (int t = 0; t < 8; ++t) dst[i + t * T] = v[t];
  }
  for (; i < end; i += T) dst[i] = src[i];
}

// streaming read: every thread folds its 16-byte words into one and stores it, so nothing is elided
__global__ __launch_bounds__(256) void read_probe(const uint4* src, size_t n16, uint32_t* sink) {
  size_t begin, end;
  probe_slab(n16, begin, end);
  const size_t T = blockDim.x;
  uint32_t acc = 0;
  size_t i = begin + threadIdx.x;
  auto fold = [&](const uint4 (&v)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t) acc ^= v[t].x ^ v[t].y ^ v[t].z ^ v[t].w;
  };
  if (i + 7 * T < end) {
    uint4 va[8], vb[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) va[t] = load16(src + i + t * T);
    i += 8 * T;
    for (; i + 15 * T < end; i += 16 * T) {
#pragma unroll
      for (int t = 0; t < 8; ++t) vb[t] = load16(src + i + t * T);
      fold(va);
#pragma unroll
      for (int t = 0; t < 8; ++t) va[t] = load16(src + i + (8 + t) * T);
      fold(vb);
    }
    fold(va);
  }
  for (; i < end; i += T) {
    const uint4 v = src[i];
    acc ^= v.x ^ v.y ^ v.z ^ v.w;
  }
  sink[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = acc;
}

__global__ void clear_words(int32_t* w, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) w[i] = 0;
}

template <class T, int DH>
hipError_t launch_rows_dh(const AppendArgs& args, hipStream_t s) {
  AppendArgs a = args;
  const int64_t heads = (int64_t)a.B * a.H_kv;
  if (a.tiled) {
    hipLaunchKernelGGL((append_rows_tiled<T, DH>), dim3(heads), dim3(BT), 0, s, a);
  } else {
    const AppendSplit plan = append_split(heads, a.n_new, DH, (int64_t)(a.scratch_bytes / (heads * (DH * sizeof(double) + sizeof(int2)))));
    const int64_t n = plan.n_split;
    a.n_split = plan.n_split; a.tiles_per_split = plan.tiles_per_split;
    a.part_ws = reinterpret_cast<double*>(a.scratch);
    a.span_ws = reinterpret_cast<int2*>(a.part_ws + (n > 1 ? heads * n * DH : 0));
    if (heads * n > kAppendOneLaunch || heads + a.B > kTickets) a.tickets = nullptr;
    if (!a.tickets && append_short(heads, a.n_new, DH)) {
      a.n_split = 1;
      hipLaunchKernelGGL((append_rows_short<T, DH>), dim3(heads), dim3(BT), 0, s, a);
    } else {
      hipLaunchKernelGGL((append_rows<T, DH>), dim3(heads * n), dim3(BT), 0, s, a);
    }
    if (a.tickets) return hipGetLastError();
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (!a.tiled && a.n_split > 16) hipLaunchKernelGGL((append_finish<DH, 1024>), dim3(heads), dim3(1024), 0, s, a);
  else if (!a.tiled && a.n_split > 1) hipLaunchKernelGGL((append_finish<DH, BT>), dim3(heads), dim3(BT), 0, s, a);
  else hipLaunchKernelGGL(bump_seq_lens, dim3((a.B + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <class T>
hipError_t launch_rows(const AppendArgs& a, hipStream_t s) {
  switch (a.d_h) {
    case 64:  return launch_rows_dh<T, 64>(a, s);
    case 128: return launch_rows_dh<T, 128>(a, s);
    case 256: return launch_rows_dh<T, 256>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

size_t append_scratch_bytes(int64_t heads, int S_max, int d_h) {
  const int64_t positions = append_tile(d_h), tiles = (S_max + 63 + positions - 1) / positions;
  int64_t n = kAppendGroups / heads + 1;           // append_groups of any number of tiles up to these
  n = n < tiles ? n : tiles;
  n = n < 128 ? n : 128;
  return n > 1 ? (size_t)heads * n * (d_h * sizeof(double) + sizeof(int2)) : 0;
}

hipError_t launch_append(const AppendArgs& a, int dtype, hipStream_t s) {
  if (a.n_new == 1) {
    if (a.tiled) {
      if (dtype == 1) hipLaunchKernelGGL(append_one_row_tiled<BF16>, dim3(a.B), dim3(512), 0, s, a);
      else hipLaunchKernelGGL(append_one_row_tiled<F16>, dim3(a.B), dim3(512), 0, s, a);
    } else if (dtype == 1) hipLaunchKernelGGL(append_one_row<BF16>, dim3(a.B), dim3(512), 0, s, a);
    else hipLaunchKernelGGL(append_one_row<F16>, dim3(a.B), dim3(512), 0, s, a);
    return hipGetLastError();
  }
  return dtype == 1 ? launch_rows<BF16>(a, s) : launch_rows<F16>(a, s);
}

hipError_t launch_copy_probe(void* dst, const void* src, size_t n_bytes, hipStream_t s) {
  hipLaunchKernelGGL(copy_probe, dim3(kProbeBlocks), dim3(256), 0, s, reinterpret_cast<uint4*>(dst),
                     reinterpret_cast<const uint4*>(src), n_bytes / 16);
  return hipGetLastError();
}

hipError_t launch_read_probe(const void* src, size_t n_bytes, void* sink, hipStream_t s) {
  hipLaunchKernelGGL(read_probe, dim3(kProbeBlocks), dim3(256), 0, s, reinterpret_cast<const uint4*>(src),
                     n_bytes / 16, reinterpret_cast<uint32_t*>(sink));
  return hipGetLastError();
}

hipError_t launch_clear(void* workspace, int n_bytes, hipStream_t s) {
  hipLaunchKernelGGL(clear_words, dim3(1), dim3(256), 0, s, reinterpret_cast<int32_t*>(workspace), n_bytes / 4);
  return hipGetLastError();
}

}  // namespace sparq
