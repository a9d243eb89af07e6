// Commit of verified rows to the paged KV cache (Sec. 4.3, decoupled execution: the cache
// written by target verification is what the next draft step reuses).
//
// One work-group per sequence, one launch: every wave reads the sequence's length, the work-group copies
// new rows 0 .. accept_len (K and V, all KV heads, 16-byte accesses) to logical positions
// kv_len + j, and, past a barrier, writes the new length last -- so the output array may be the input array.  Only
// verify rows are ever written: mask tokens stay invisible to the clean prefix (Sec. 4.1), so a
// sequence without verify rows commits nothing and accept_len is held below the number of verify rows.
#include "fd_common.h"

namespace fd {

constexpr int AT_ONCE = 4;

template <typename T>
__global__ __launch_bounds__(256) void append_kv_kernel(AttnParams p, T* __restrict__ k_cache, T* __restrict__ v_cache,
                                                        const int* __restrict__ accept_len, int* __restrict__ kv_len_out) {
  const int seq = blockIdx.x;
  const int accepted = sload(accept_len, seq);                // (requested with the lengths)
  const SeqInfo s = load_seq(p, seq);                         // clamps and reports bad lengths; reads kv_len[seq]
  int rows = 0;                                               // rows this sequence commits
  if (s.k > 0) {
    int acc = accepted;
    if (acc < 0 || acc >= s.k) { if (threadIdx.x == 0) flag_status(p.status, FD_DEV_ROWS_RANGE); acc = clampi(acc, 0, s.k - 1); }
    rows = acc + 1;
    // kv_len is the length BEFORE the commit; load_seq checked that the page list covers it, the rows
    // added here need their own check: whatever the list has no room for is not committed
    const int room = s.npages * p.page_size - s.L;
    if (rows > room) { if (threadIdx.x == 0) flag_status(p.status, FD_DEV_PAGE_RANGE); rows = room < 0 ? 0 : room; }
  }
  constexpr int VEC = 16 / sizeof(T);                          // elements per 16-byte vector
  const int vec_per_head = p.D / VEC;                          // head_dim is a multiple of 8
  const int nvec = p.Hkv * vec_per_head;
  // AT_ONCE rows of a thread's vector are in flight together with their page ids, which only the stores need: row by row, with
  // the page first, each row was two latencies of memory (a few rows of 8 heads of 128: kernel 4.1 -> 3.0 us, a step of four layers 107.2 -> 105.1).
  const int lp0 = s.L / p.page_size, slot0 = s.L - lp0 * p.page_size;
  for (int i = threadIdx.x; i < 2 * nvec; i += 256) {
    const bool is_v = i >= nvec;
    const int iv = is_v ? i - nvec : i;
    const int h = iv / vec_per_head, e = (iv - h * vec_per_head) * VEC;
    const T* src = reinterpret_cast<const T*>(is_v ? p.v_new : p.k_new) + (long long)s.row0 * p.Hkv * p.D + h * p.D + e;
    T* dst = (is_v ? v_cache : k_cache) + (long long)h * p.sh + e;
    int lp = lp0, slot = slot0;
    for (int j0 = 0; j0 < rows; j0 += AT_ONCE) {
      u32x4 val[AT_ONCE]; int phys[AT_ONCE], at[AT_ONCE];
#pragma unroll
      for (int u = 0; u < AT_ONCE; ++u) {
        const bool there = j0 + u < rows;          // (uniform)
        phys[u] = -1; at[u] = slot;
        if (there) {
          phys[u] = sload(p.page_indices, s.page0 + lp);
          val[u] = *reinterpret_cast<const u32x4*>(src + (long long)(j0 + u) * p.Hkv * p.D);
          if (++slot == p.page_size) { slot = 0; ++lp; }
        }
      }
#pragma unroll
      for (int u = 0; u < AT_ONCE; ++u) {
        if (j0 + u >= rows) break;
        if (phys[u] < 0 || phys[u] >= p.num_pages) { if (i == 0) flag_status(p.status, FD_DEV_PAGE_RANGE); continue; }
        *reinterpret_cast<u32x4*>(dst + (long long)phys[u] * p.sp + (long long)at[u] * p.st) = val[u];
      }
    }
  }
  // The output may be the input array, and each of the four waves reads the old length for itself: the new one waits until
  // all of them have used it.  No other work-group reads kv_len[seq].
  __syncthreads();
  if (threadIdx.x == 0) kv_len_out[seq] = s.L + rows;
}

hipError_t run_append_kv(const AttnParams& p, int dtype, void* k_cache, void* v_cache, const int* accept_len,
                         int* kv_len_out, hipStream_t st) {
  if (dtype == FD_BF16)
    hipLaunchKernelGGL(append_kv_kernel<bf16_t>, dim3(p.B), dim3(256), 0, st, p, reinterpret_cast<bf16_t*>(k_cache),
                       reinterpret_cast<bf16_t*>(v_cache), accept_len, kv_len_out);
  else
    hipLaunchKernelGGL(append_kv_kernel<float>, dim3(p.B), dim3(256), 0, st, p, reinterpret_cast<float*>(k_cache),
                       reinterpret_cast<float*>(v_cache), accept_len, kv_len_out);
  return hipGetLastError();
}

}  // namespace fd
