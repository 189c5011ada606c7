// Closing a verification round: the window's new K/V rows are appended to the
// paged cache, and each request's accepted length is committed.
//
// The cache is append-dominant: an iteration only adds the K/V of the tokens
// it processed (Section 3).  Request r's window (anchor + K_r proposals) sits
// at positions L_r - n_q .. L_r - 1; token t lives in slot t % 16 of block
// block_table[r][t / 16].  After acceptance the request keeps its anchor and
// its n_r accepted proposals: L'_r = L_r - K_r + n_r (the resampled or bonus
// token is the next round's anchor).
//
// kv_append: one workgroup per (KV head, request, layer).  Memory writes whole
// 32-byte sectors cheaply and partial ones with a read-modify-write in the
// memory system, which also delays the kernels that follow (a decode
// attention launched right after an append made of 2-byte element stores
// ran 6 % slower).  So the kernel writes whole sectors only: for every block
// the window touches, thread t < head_dim rewrites dimension t's 16-slot V row
// (32 bytes) and, as (run c, slot pair), the two 16-byte K runs of a slot pair
// that the window touches, taking the window's slots from the new rows and every
// other slot from the sector's current contents.  Only this workgroup writes the
// (block, KV head) tile, so the merge needs no ordering.  Volume: the
// sectors the window touches, read and written (about 4.5 KiB each way per
// (request, KV head) for a one-token window at head_dim 128, 13 MB each way
// for a verify_8b layer's five-token windows).
//
// Latency bounds small batches (offsets, block id, sector, store, once per block),
// so a round appends all its layers, into the pool and the staging bank, in one
// launch, and the new rows are loaded while the ids arrive.  Large ones are bound
// by the workgroups in flight, so both planes are one set of head_dim threads: a
// second set for K left most of its threads idle and a device's worth of wave
// slots short (8 KV heads, head_dim 128: one-token windows of 512 requests 14.5 us
// with it, 10.3 without, 256 requests 8.8 and 6.9; five-token windows of 256 12.6
// and 10.5, of 32 4.4 and 4.5).  Four layers of 32 requests (five-token windows,
// 10 of them staged): eight launches of 6.4 to 6.9 us -> one of 8.0 us; one layer
// of 64 requests (one token) into pool and staging bank 2 x 4.7 -> 4.2 us.
#include "nsd_internal.h"

#include <type_traits>

namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kAppendLayers = 32;   // layers of one launch (their rows are kernel arguments)

// The paged planes a window goes to, stacked over layers, and the block table
// that says where (a negative id: not here).
struct Bank {
  uint16_t* k;
  uint16_t* v;
  const int32_t* table;
  int64_t num_blocks;   // 0: no such bank
};

// LAYERS and BANKS: the most a launch takes (one layer into one bank is the
// draft step's call).
template <int LAYERS, int BANKS>
struct AppendArgs {
  Bank bank[BANKS];
  const uint16_t* k_new[LAYERS];
  const uint16_t* v_new[LAYERS];
  int32_t max_blocks_per_seq, num_kv_heads, head_dim, total_q;
  int32_t aligned;              // every k_new is 16-byte aligned
};

// Sector p of a plane: the elements at bits m become w.
__device__ inline void merge_sector(u32x4* p, u32x4 lo, u32x4 hi, const uint32_t (&w)[8],
                                    const uint32_t (&m)[8]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    lo[e] = (lo[e] & ~m[e]) | w[e];
    hi[e] = (hi[e] & ~m[4 + e]) | w[4 + e];
  }
  p[0] = lo;
  p[1] = hi;
}

template <int LAYERS, int BANKS>
__global__ __launch_bounds__(128) void kv_append_kernel(
    AppendArgs<LAYERS, BANKS> A, const int32_t* __restrict__ table0, const int32_t* __restrict__ table1,
    const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ q_indptr) {
  const int g = blockIdx.x;
  const int r = blockIdx.y;
  const int layer = LAYERS == 1 ? 0 : blockIdx.z;
  const int tid = threadIdx.x;
  const int d = A.head_dim, hkv = A.num_kv_heads;
  const int a = q_indptr[r];
  const int nq = q_indptr[r + 1] - a;
  const int L = seq_lens[r];
  if (nq <= 0) return;
  // window positions inside [0, 16 * max_blocks_per_seq)
  const int64_t t0 = max((int64_t)L - nq, (int64_t)0);
  const int64_t t1 = min((int64_t)L - 1, (int64_t)A.max_blocks_per_seq * 16 - 1);
  const int64_t row_len = (int64_t)hkv * d;
  const uint16_t* kn = A.k_new[layer] + (int64_t)g * d;
  const uint16_t* vn = A.v_new[layer] + (int64_t)g * d;
  const int runs = d / 8, c = tid % runs;
  for (int64_t blk = t0 / 16; blk <= t1 / 16 && t0 <= t1; ++blk) {
    const int64_t entry = (int64_t)r * A.max_blocks_per_seq + blk;
    const int32_t id[2] = {table0[entry], BANKS == 2 ? table1[entry] : -1};
    // the window's slots of the block; slot s takes row first + s (a row
    // outside [0, total_q) leaves its slot)
    const int64_t first = (int64_t)a + blk * 16 - ((int64_t)L - nq);
    const int s_lo = (int)max(max(t0 - blk * 16, (int64_t)0), min((int64_t)16, -first));
    const int s_hi = (int)min(min(t1 - blk * 16, (int64_t)15),
                              max((int64_t)-1, (int64_t)A.total_q - 1 - first));
    if (s_lo > s_hi) continue;
    // K: the runs of this thread's slot pair, where the window has that many pairs
    // (a load that the others skip: loaded by all, it cost one-token windows 12 %)
    const int pr = s_lo / 2 + tid / runs;
    const bool has_k = pr <= s_hi / 2;
    u32x4 x[2] = {};
    if (has_k) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint16_t* src = kn + (first + min(max(2 * pr + u, s_lo), s_hi)) * row_len + c * 8;
        if (A.aligned) {
          x[u] = *(const u32x4*)src;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) x[u][e] = src[2 * e] | (uint32_t)src[2 * e + 1] << 16;
        }
      }
    }
    // V: dimension tid's slots, w the new elements at the bits m
    uint32_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0}, m[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      m[i] = (2 * i >= s_lo && 2 * i <= s_hi ? 0xffffu : 0u) |
             (2 * i + 1 >= s_lo && 2 * i + 1 <= s_hi ? 0xffff0000u : 0u);
    auto put = [&](int s, uint32_t v) {
      const uint32_t e = v << (s % 2 * 16);
#pragma unroll
      for (int i = 0; i < 8; ++i) w[i] |= i == s / 2 ? e : 0u;   // fixed indices: registers
    };
    int s = s_lo;
    for (; s + 3 <= s_hi; s += 4) {
      uint32_t v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = vn[(first + s + u) * row_len + tid];
#pragma unroll
      for (int u = 0; u < 4; ++u) put(s + u, v[u]);
    }
    for (; s <= s_hi; ++s) put(s, vn[(first + s) * row_len + tid]);
    uint32_t kw[8], km[8];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t bits = 2 * pr + u >= s_lo && 2 * pr + u <= s_hi ? 0xffffffffu : 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        kw[u * 4 + e] = x[u][e] & bits;
        km[u * 4 + e] = bits;
      }
    }
#pragma unroll
    for (int b = 0; b < BANKS; ++b) {
      const Bank& to = A.bank[b];
      if (id[b] < 0 || id[b] >= to.num_blocks) continue;   // an invalid id is not written
      const int64_t tile = (((int64_t)layer * to.num_blocks + id[b]) * hkv + g) * d * 16;
      u32x4* vp = (u32x4*)(to.v + tile + (int64_t)tid * 16);
      u32x4* kp = (u32x4*)(to.k + tile + (int64_t)(c * 16 + 2 * pr) * 8);
      const u32x4 v0 = vp[0], v1 = vp[1];
      u32x4 k0 = {}, k1 = {};
      if (has_k) {
        k0 = kp[0];
        k1 = kp[1];
      }
      merge_sector(vp, v0, v1, w, m);
      if (has_k) merge_sector(kp, k0, k1, kw, km);
    }
  }
}

__global__ __launch_bounds__(256) void commit_kernel(const int32_t* __restrict__ seq_lens,
                                                     const int32_t* __restrict__ q_indptr,
                                                     const int32_t* __restrict__ accepted_len,
                                                     int32_t* __restrict__ new_lens, int32_t bs) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= bs) return;
  const int k = max(0, q_indptr[r + 1] - q_indptr[r] - 1);
  const int n = min(max(accepted_len[r], 0), k);
  new_lens[r] = seq_lens[r] - k + n;
}

}  // namespace

static nsd_status append_layers(const char* fn, const Bank* banks, int32_t n_layers,
                                const void* const* k_new, const void* const* v_new,
                                int32_t max_blocks_per_seq, const int32_t* seq_lens,
                                const int32_t* q_indptr, int32_t bs, int32_t total_q,
                                int32_t num_kv_heads, int32_t block_size, int32_t head_dim,
                                void* stream) {
  using namespace nsd;
  const bool second = banks[1].table && banks[1].num_blocks > 0;
  if (block_size != NSD_BLOCK_SIZE)
    return fail(NSD_ERR_UNSUPPORTED, "%s: block_size must be 16 (got %d)", fn, block_size);
  if (head_dim != 64 && head_dim != 128)
    return fail(NSD_ERR_UNSUPPORTED, "%s: head_dim must be 64 or 128 (got %d)", fn, head_dim);
  if (bs < 0 || total_q < 0 || num_kv_heads < 1 || num_kv_heads > 65535 || bs > 65535 ||
      max_blocks_per_seq < 1 || banks[0].num_blocks < 0 || banks[1].num_blocks < 0 || n_layers < 0)
    return fail(NSD_ERR_SHAPE, "%s: bad sizes", fn);
  // planes stacked over layers are addressed with 64-bit byte offsets
  for (int b = 0; b < 2; ++b) {
    int64_t bytes;
    if (n_layers > 1 &&
        (__builtin_mul_overflow(banks[b].num_blocks, (int64_t)num_kv_heads * head_dim * 32, &bytes) ||
         __builtin_mul_overflow(bytes, (int64_t)n_layers, &bytes)))
      return fail(NSD_ERR_SHAPE, "%s: planes of more than 2^63-1 bytes", fn);
  }
  if (bs == 0 || total_q == 0 || n_layers == 0) return NSD_OK;
  if (!banks[0].k || !banks[0].v || !k_new || !v_new || !banks[0].table || !seq_lens ||
      !q_indptr || (second && (!banks[1].k || !banks[1].v)))
    return fail(NSD_ERR_NULL, "%s: NULL pointer argument", fn);
  for (int l = 0; l < n_layers; ++l)
    if (!k_new[l] || !v_new[l]) return fail(NSD_ERR_NULL, "%s: NULL pointer argument", fn);
  if (((uintptr_t)banks[0].k | (uintptr_t)banks[0].v) % 16)
    return fail(NSD_ERR_SHAPE, "%s: k_pool and v_pool must be 16-byte aligned", fn);
  if (second && ((uintptr_t)banks[1].k | (uintptr_t)banks[1].v) % 16)
    return fail(NSD_ERR_SHAPE, "%s: k_stage and v_stage must be 16-byte aligned", fn);
  clear_stale_error();
  for (int l0 = 0; l0 < n_layers; l0 += kAppendLayers) {
    const int n = n_layers - l0 < kAppendLayers ? n_layers - l0 : kAppendLayers;
    auto go = [&](auto layers, auto bank_count) {
      constexpr int kLayers = decltype(layers)::value, kBanks = decltype(bank_count)::value;
      AppendArgs<kLayers, kBanks> A;
      for (int b = 0; b < kBanks; ++b) {
        A.bank[b] = b == 0 || second ? banks[b] : Bank{nullptr, nullptr, nullptr, 0};
        const int64_t before = l0 * A.bank[b].num_blocks * num_kv_heads * head_dim * 16;
        A.bank[b].k += before;
        A.bank[b].v += before;
      }
      A.aligned = 1;
      for (int l = 0; l < kLayers; ++l) {
        A.k_new[l] = l < n ? (const uint16_t*)k_new[l0 + l] : nullptr;
        A.v_new[l] = l < n ? (const uint16_t*)v_new[l0 + l] : nullptr;
        if ((uintptr_t)A.k_new[l] % 16) A.aligned = 0;
      }
      A.max_blocks_per_seq = max_blocks_per_seq;
      A.num_kv_heads = num_kv_heads;
      A.head_dim = head_dim;
      A.total_q = total_q;
      hipLaunchKernelGGL((kv_append_kernel<kLayers, kBanks>), dim3(num_kv_heads, bs, n),
                         dim3(head_dim), 0, (hipStream_t)stream, A, banks[0].table,
                         second ? banks[1].table : banks[0].table, seq_lens, q_indptr);
    };
    if (n_layers == 1 && !second)
      go(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{});
    else
      go(std::integral_constant<int, kAppendLayers>{}, std::integral_constant<int, 2>{});
  }
  return check_launch(fn);
}

extern "C" nsd_status nsd_kv_append(void* k_pool, void* v_pool, int64_t num_blocks,
                                    const void* k_new, const void* v_new,
                                    const int32_t* block_table, int32_t max_blocks_per_seq,
                                    const int32_t* seq_lens, const int32_t* q_indptr,
                                    int32_t bs, int32_t total_q, int32_t num_kv_heads,
                                    int32_t block_size, int32_t head_dim, void* stream) {
  const Bank banks[2] = {{(uint16_t*)k_pool, (uint16_t*)v_pool, block_table, num_blocks},
                         {nullptr, nullptr, nullptr, 0}};
  return append_layers("kv_append", banks, 1, &k_new, &v_new, max_blocks_per_seq, seq_lens,
                       q_indptr, bs, total_q, num_kv_heads, block_size, head_dim, stream);
}

extern "C" nsd_status nsd_kv_append_layers(
    void* k_pool, void* v_pool, int64_t num_blocks, const int32_t* block_table, void* k_stage,
    void* v_stage, int64_t stage_num_blocks, const int32_t* stage_rows, int32_t n_layers,
    const void* const* k_new, const void* const* v_new, int32_t max_blocks_per_seq,
    const int32_t* seq_lens, const int32_t* q_indptr, int32_t bs, int32_t total_q,
    int32_t num_kv_heads, int32_t block_size, int32_t head_dim, void* stream) {
  const Bank banks[2] = {
      {(uint16_t*)k_pool, (uint16_t*)v_pool, block_table, num_blocks},
      {(uint16_t*)k_stage, (uint16_t*)v_stage, stage_rows, stage_rows ? stage_num_blocks : 0}};
  return append_layers("kv_append_layers", banks, n_layers, k_new, v_new, max_blocks_per_seq,
                       seq_lens, q_indptr, bs, total_q, num_kv_heads, block_size, head_dim,
                       stream);
}

extern "C" nsd_status nsd_commit_lengths(const int32_t* seq_lens, const int32_t* q_indptr,
                                         const int32_t* accepted_len, int32_t* new_lens,
                                         int32_t bs, void* stream) {
  using namespace nsd;
  const char* fn = "commit_lengths";
  if (bs < 0) return fail(NSD_ERR_SHAPE, "%s: bs < 0", fn);
  if (bs == 0) return NSD_OK;
  if (!seq_lens || !q_indptr || !accepted_len || !new_lens)
    return fail(NSD_ERR_NULL, "%s: NULL pointer argument", fn);
  clear_stale_error();
  hipLaunchKernelGGL(commit_kernel, dim3((uint32_t)(((int64_t)bs + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream,
                     seq_lens, q_indptr, accepted_len, new_lens, bs);
  return check_launch(fn);
}

extern "C" nsd_status nsd_host_alias(const void* host, void** device_alias) {
  using namespace nsd;
  if (!host || !device_alias) return fail(NSD_ERR_NULL, "host_alias: NULL pointer argument");
  hipPointerAttribute_t a;
  if (hipPointerGetAttributes(&a, host) != hipSuccess || a.type != hipMemoryTypeHost ||
      !a.devicePointer) {
    (void)hipGetLastError();
    return fail(NSD_ERR_UNSUPPORTED, "host_alias: not pinned host memory mapped for the device");
  }
  // the alias of the allocation base, shifted to this pointer
  *device_alias = (char*)a.devicePointer + ((const char*)host - (const char*)a.hostPointer);
  return NSD_OK;
}
