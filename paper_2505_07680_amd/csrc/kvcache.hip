// KV-cache state updates around the verify step (Section 4.4, StateManager):
//
//   kv_append:  a step's gamma_b + 1 new K/V rows (the pending token and the
//               drafts) written at the sequence's cursor and marked valid.
//               The cursor is the sequence's own length, or one physical
//               length shared by the batch (the paper's layout: a sequence
//               that rolled back further keeps masked holes below it).
//   kv_compact: optional reclamation of the holes: each sequence's valid
//               rows moved to the front in order (in place), then the mask
//               and length rewritten.
//
// K/V bytes move verbatim (16-byte vector loads and stores).

#include "sr_internal.h"

namespace sr {
namespace {

constexpr int kKvThreads = 256;

// One workgroup per sequence: the cursor is read once, every row chunk is
// copied, then the length is advanced (the only writer of kv_len[b]). Bound by
// latency: every thread has kAppendUnroll chunks of K and of V in flight (one
// chunk each in 256 threads took 6.3 us for 7 rows of 32 heads of 128, now
// 4.6).
constexpr int kAppendThreads = 1024;
constexpr int kAppendUnroll = 4;
__global__ void __launch_bounds__(kAppendThreads)
kv_append_kernel(const u32x4* __restrict__ k_new, const u32x4* __restrict__ v_new,
                 const int32_t* __restrict__ gamma, u32x4* __restrict__ k_cache, u32x4* __restrict__ v_cache,
                 uint8_t* __restrict__ mask, int32_t* __restrict__ kv_len, const int32_t* __restrict__ shared_len,
                 int gmax, int Hkv, int D, int L_cap, int32_t* __restrict__ status) {
  __shared__ int s_cur, s_n;
  const int b = blockIdx.x;
  if (threadIdx.x == 0) {
    const int g = gamma[b];
    const int L = kv_len[b];
    const int cur = shared_len ? *shared_len : L;
    int n = g + 1;
    uint32_t bad = 0;
    if (g < 0 || g > gmax) bad |= SR_ST_GAMMA;
    else if (L < 0 || L > L_cap || cur < 0 || cur + n > L_cap) bad |= SR_ST_KVLEN;
    if (bad) {
      n = 0;
      if (status) atomicOr(status, (int32_t)bad);
    }
    s_cur = cur;
    s_n = n;
  }
  __syncthreads();
  const int cur = s_cur, n = s_n;
  const int cpr = D / 8;  // 16-byte chunks per row
  const int total = n * Hkv * cpr;
  const u32x4* ks = k_new + (size_t)b * (gmax + 1) * Hkv * cpr;  // the new rows are one run
  const u32x4* vs = v_new + (size_t)b * (gmax + 1) * Hkv * cpr;
  for (int i0 = threadIdx.x; i0 < total; i0 += kAppendThreads * kAppendUnroll) {
    u32x4 kr[kAppendUnroll], vr[kAppendUnroll];
#pragma unroll
    for (int u = 0; u < kAppendUnroll; ++u) {
      const int idx = min(i0 + u * kAppendThreads, total - 1);
      kr[u] = ks[idx];
      vr[u] = vs[idx];
    }
#pragma unroll
    for (int u = 0; u < kAppendUnroll; ++u) {
      const int idx = i0 + u * kAppendThreads;
      if (idx < total) {
        const int c = idx % cpr;
        const int h = (idx / cpr) % Hkv;
        const int i = idx / (cpr * Hkv);
        const size_t dst = (((size_t)b * Hkv + h) * L_cap + cur + i) * cpr + c;
        k_cache[dst] = kr[u];
        v_cache[dst] = vr[u];
      }
    }
  }
  if (mask)
    for (int i = threadIdx.x; i < n; i += kAppendThreads) mask[(size_t)b * L_cap + cur + i] = 1;
  if (threadIdx.x == 0 && n > 0) kv_len[b] = cur + n;
}

// Compaction of one K or V slab of a (sequence, kv head), in place. One wave
// per slab and 128-byte column of its rows (whole cache lines: columns of 64 or
// 32 bytes, for more waves, wrote partial lines and were slower than one
// workgroup per slab), 128 positions per block, so no wave waits for another. A
// block's valid rows move to off, off + 1, ... (off: the valid rows before it),
// never up. Two blocks are in flight: the next block's loads are issued before
// this block's stores, whose rows all lie below it, and a block is stored only
// when all its loads have returned, so no row is overwritten before it has been
// read. Blocks whose rows all stay are neither read nor written.
//
// Bound by HBM, reads and writes in equal parts. With one workgroup per slab
// that moved 64 whole rows per round trip (load, wait, barrier, store), 32
// sequences of 2048 to 4096 rows with 2% holes (8 heads x 128) took 267 us; now
// 164 (4.8 TB/s, a device copy reaches 5.0). Two slabs of 32768 rows each:
// 1747 to 254 us.
constexpr int kCompactBlock = 128;

template <int D>
__global__ void __launch_bounds__(64)
kv_compact_kernel(u32x4* __restrict__ k_cache, u32x4* __restrict__ v_cache, const uint8_t* __restrict__ mask,
                  const int32_t* __restrict__ kv_len, int Hkv, int L_cap) {
  constexpr int kRow = D * 2;               // bytes per row
  constexpr int kLanes = 8;                 // lanes per row: 128 bytes
  constexpr int kCols = kRow / 128;
  constexpr int kRows = 64 / kLanes;        // rows per load
  constexpr int kLoads = kCompactBlock / kRows;
  constexpr uint32_t kOut = 0x7ffffff0u;    // past every resource: reads zero, stores nothing
  constexpr int kStream = 2;                // cache-policy operand: non-temporal
  const unsigned slab = blockIdx.x / (2 * kCols);  // (sequence, kv head)
  const unsigned part = blockIdx.x % (2 * kCols);  // K or V, and the column
  const int b = (int)(slab / (unsigned)Hkv);
  const int L = kv_len[b];
  if (L < 0 || L > L_cap) return;           // reported by the mask kernel
  const int lane = threadIdx.x;
  const int lrow = lane / kLanes;
  const uint32_t col = (uint32_t)(((part / 2) * kLanes + lane % kLanes) * 16);
  char* base = (char*)((part & 1) ? v_cache : k_cache) + (size_t)slab * L_cap * kRow;
  // the mask row as a resource from the aligned word at or below its start
  const uint8_t* mrow = mask + (size_t)b * L_cap;
  const uint32_t skew = (uint32_t)((uintptr_t)mrow & 3);
  const __amdgpu_buffer_rsrc_t rm = make_rsrc(mrow - skew, (size_t)L + skew);

  struct Block {
    u32x4 r[kLoads];
    uint64_t lo, hi;  // valid rows
    int at, off;      // first position; where its valid rows go
    bool move;
  };
  // the mask bytes of a block (0 past the length)
  struct MaskBytes {
    uint8_t lo, hi;
  };
  auto fetch_mask = [&](int at) __attribute__((always_inline)) {
    MaskBytes m;
    m.lo = __builtin_amdgcn_raw_buffer_load_b8(rm, skew + (uint32_t)(at + lane), 0, 0);
    m.hi = __builtin_amdgcn_raw_buffer_load_b8(rm, skew + (uint32_t)(at + 64 + lane), 0, 0);
    return m;
  };
  // row u * kRows + lrow of a block: valid, and how many valid rows of the block precede it
  auto rank = [&](const Block& B, int u, bool& valid) __attribute__((always_inline)) {
    const bool upper = u * kRows >= 64;  // (compile-time: a load's rows lie in one word)
    const uint64_t word = upper ? B.hi : B.lo;
    const int p = u * kRows + lrow - (upper ? 64 : 0);
    valid = ((word >> p) & 1ull) != 0ull;
    return (upper ? (int)__popcll(B.lo) : 0) + (int)__popcll(word & ((1ull << p) - 1ull));
  };
  int off = 0;  // valid rows before the next block to load
  auto load = [&](Block& B, int at, const MaskBytes& m) __attribute__((always_inline)) {
    B.lo = __ballot(m.lo != 0);
    B.hi = __ballot(m.hi != 0);
    B.at = at;
    B.off = off;
    const int n = (int)__popcll(B.lo) + (int)__popcll(B.hi);
    // rows stay where they are while there has been no hole (n counts every position up to the length)
    B.move = at < L && !(off == at && n == min(kCompactBlock, L - at));
    off += n;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(base + (size_t)at * kRow, B.move ? (size_t)kCompactBlock * kRow : 0);
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      bool valid;
      rank(B, u, valid);
      const uint32_t o = valid ? (uint32_t)((u * kRows + lrow) * kRow) + col : kOut;
      B.r[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, kStream));
    }
  };
  auto store = [&](Block& B) __attribute__((always_inline)) {
    if (!B.move) return;  // wave-uniform
    // every load of the block has returned before any store
#pragma unroll
    for (int u = 0; u < kLoads; ++u) asm volatile("" : "+v"(B.r[u])::"memory");
    __builtin_amdgcn_sched_barrier(0);
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(base + (size_t)B.off * kRow, (size_t)kCompactBlock * kRow);
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      bool valid;
      const int k = rank(B, u, valid);
      const uint32_t o = valid ? (uint32_t)(k * kRow) + col : kOut;
      __builtin_amdgcn_raw_buffer_store_b128(B.r[u], rs, o, 0, kStream);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  Block x, y;
  MaskBytes m0 = fetch_mask(0), m1 = fetch_mask(kCompactBlock);
  load(x, 0, m0);
  for (int at = 0; at < L; at += 2 * kCompactBlock) {
    m0 = fetch_mask(at + 2 * kCompactBlock);
    load(y, at + kCompactBlock, m1);
    __builtin_amdgcn_sched_barrier(0);
    store(x);
    m1 = fetch_mask(at + 3 * kCompactBlock);
    load(x, at + 2 * kCompactBlock, m0);
    __builtin_amdgcn_sched_barrier(0);
    store(y);
  }
}

// After every slab of a sequence moved: mask = 1 on the new prefix, 0 up to
// the old length; kv_len = the count of valid rows. Four bytes per access (the
// mask row's start need not be aligned: the resource starts at the aligned
// word below it, and the bytes outside the row keep what they hold).
__global__ void __launch_bounds__(kKvThreads)
kv_compact_mask_kernel(uint8_t* __restrict__ mask, int32_t* __restrict__ kv_len, int L_cap,
                       int32_t* __restrict__ status) {
  __shared__ int s_part[kKvThreads / 64];
  const int b = blockIdx.x;
  const int L = kv_len[b];
  if (L < 0 || L > L_cap) {
    if (threadIdx.x == 0 && status) atomicOr(status, (int32_t)SR_ST_KVLEN);
    return;
  }
  uint8_t* row = mask + (size_t)b * L_cap;
  // whole aligned words [w0, w1) of the row, and the bytes before and after them
  const int head = min((int)((4 - ((uintptr_t)row & 3)) & 3), L);
  const int words = (L - head) / 4;
  uint32_t* wrow = (uint32_t*)(row + head);
  const int tid = threadIdx.x;
  int cnt = 0;
  constexpr int kU = 4;
  for (int i0 = 0; i0 < words; i0 += kKvThreads * kU) {
    uint32_t x[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = i0 + u * kKvThreads + tid;
      x[u] = i < words ? wrow[i] : 0u;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u)  // non-zero bytes
      cnt += ((x[u] & 0xffu) != 0u) + ((x[u] & 0xff00u) != 0u) + ((x[u] & 0xff0000u) != 0u) + ((x[u] & 0xff000000u) != 0u);
  }
  const int tail = head + words * 4;
  if (tid < head) cnt += row[tid] != 0;
  if (tid < L - tail) cnt += row[tail + tid] != 0;
  const int w = wave_id();
  const int tot = wave_incl_scan_i(cnt);
  if ((tid & 63) == 63) s_part[w] = tot;
  __syncthreads();
  int n = 0;
  for (int i = 0; i < kKvThreads / 64; ++i) n += s_part[i];
  // (every count is read before the mask changes: the barrier above)
  for (int i = tid; i < words; i += kKvThreads) {
    const int p = n - (head + i * 4);  // ones among the word's bytes
    wrow[i] = p >= 4 ? 0x01010101u : p <= 0 ? 0u : 0x01010101u & ((1u << (8 * p)) - 1u);
  }
  if (tid < head) row[tid] = tid < n ? 1 : 0;
  if (tid < L - tail) row[tail + tid] = tail + tid < n ? 1 : 0;
  if (tid == 0) kv_len[b] = n;
}

}  // namespace

int launch_kv_append(const void* k_new, const void* v_new, const int32_t* gamma, void* k_cache, void* v_cache,
                     uint8_t* cache_mask, int32_t* kv_len, const int32_t* shared_len, int B, int gamma_max,
                     int Hkv, int D, int L_cap, int32_t* status, hipStream_t stream) {
  hipLaunchKernelGGL(kv_append_kernel, dim3(B), dim3(kAppendThreads), 0, stream, (const u32x4*)k_new,
                     (const u32x4*)v_new, gamma, (u32x4*)k_cache, (u32x4*)v_cache, cache_mask, kv_len, shared_len,
                     gamma_max, Hkv, D, L_cap, status);
  return hipGetLastError() == hipSuccess ? SR_OK : SR_ELAUNCH;
}

int launch_kv_compact(void* k_cache, void* v_cache, uint8_t* cache_mask, int32_t* kv_len, int B, int Hkv, int D,
                      int L_cap, int32_t* status, hipStream_t stream) {
  const auto kernel = D == 64 ? kv_compact_kernel<64> : kv_compact_kernel<128>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(B * Hkv) * 2u * (unsigned)(D / 64)), dim3(64), 0, stream, (u32x4*)k_cache,
                     (u32x4*)v_cache, (const uint8_t*)cache_mask, (const int32_t*)kv_len, Hkv, L_cap);
  if (hipGetLastError() != hipSuccess) return SR_ELAUNCH;
  hipLaunchKernelGGL(kv_compact_mask_kernel, dim3(B), dim3(kKvThreads), 0, stream, cache_mask, kv_len, L_cap,
                     status);
  return hipGetLastError() == hipSuccess ? SR_OK : SR_ELAUNCH;
}

}  // namespace sr
