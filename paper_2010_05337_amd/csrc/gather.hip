// Feature-row gather on gfx950: out[i, :] = feats[ids[i], :] (the trainer's
// pull of the mini-batch's vertex features from the key-value store,
// DistDGL Section III-C, here a local copy in HBM).
//
// A group of G lanes copies one row in 16-byte chunks (shorter accesses only
// for rows below 16 bytes); every group keeps U rows in flight before it
// stores, so each wave has U independent row reads outstanding.  Rows need no
// alignment (global accesses may be misaligned), and the last chunk of a row
// that 16 does not divide starts 16 bytes before the row's end: it rewrites
// bytes of the chunk before it with the same values.  A row of 75 fp32 is so
// 19 chunks of one pass of 32 lanes; 4-byte accesses took two passes of 64.
#include "common.hpp"
#include "kernels.hpp"

#ifndef GMB_GATHER_MAX_BLOCKS
#define GMB_GATHER_MAX_BLOCKS 8192
#endif

namespace gmb {

namespace {

template <typename V>
__device__ __forceinline__ void opaque_vec(V& x) {
  static_assert(sizeof(V) % 4 == 0 || sizeof(V) == 2, "element size");
  if constexpr (sizeof(V) == 16) {
    asm volatile("" : "+v"(x.x), "+v"(x.y), "+v"(x.z), "+v"(x.w));
  } else if constexpr (sizeof(V) == 8) {
    asm volatile("" : "+v"(x.x), "+v"(x.y));
  } else {
    asm volatile("" : "+v"(x));
  }
}

// Every load is unconditional from a clamped address (row 0 for a lane
// without a row, an out-of-range id reads row 0 and is zeroed after the
// whole batch has been issued): a load under a divergent branch makes the
// compiler drain every outstanding load before the next one.
// EVEN: the row is whole chunks, and its address takes 32-bit factors and no
// select for the last chunk (half the multiplies; 346k rows of 400 bytes
// 66.2 us a call, 66.35 in the general form).
template <typename V, int G, int U, bool EVEN>
__global__ __launch_bounds__(256) void k_gather(const int32_t* __restrict__ ids, const int32_t* n_dev,
                                                int64_t n_cap, const char* __restrict__ feats,
                                                int64_t num_nodes, int64_t row_bytes, char* __restrict__ out,
                                                uint32_t* status) {
  const int cpr = static_cast<int>((row_bytes + sizeof(V) - 1) / sizeof(V));
  int64_t n = n_cap;
  if (n_dev) {
    const int32_t m = load_size(n_dev);
    n = m < 0 ? 0 : (m < n_cap ? m : n_cap);
  }
  constexpr int kGroups = 256 / G;
  const int lane = threadIdx.x & (G - 1);
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kGroups;
  bool bad = false;
  for (int64_t row = static_cast<int64_t>(blockIdx.x) * kGroups + threadIdx.x / G; row < n;
       row += stride * U) {
    int32_t id[U];
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t r = row + u * stride;
      id[u] = ids[r < n ? r : 0];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t r = row + u * stride;
      const bool ok = valid_vertex(id[u], num_nodes);
      bad |= (r < n) & !ok;
      in[u] = (r < n) & ok;
      id[u] = in[u] ? id[u] : 0;
    }
    for (int c = lane; c < cpr; c += G) {
      const int64_t at = EVEN || c + 1 < cpr ? static_cast<int64_t>(c) * sizeof(V) : row_bytes - static_cast<int64_t>(sizeof(V));
      V val[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        __builtin_memcpy(&val[u], feats + (EVEN ? (static_cast<int64_t>(id[u]) * cpr + c) * sizeof(V)
                                                : static_cast<int64_t>(id[u]) * row_bytes + at), sizeof(V));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        opaque_vec(val[u]);
        const int64_t r = row + u * stride;
        const V x = in[u] ? val[u] : V{};
        if (r < n)
          __builtin_memcpy(out + (EVEN ? (r * cpr + c) * sizeof(V) : r * row_bytes + at), &x, sizeof(V));
      }
    }
  }
  if (bad) raise_status(status, GMB_STATUS_ERANGE);
}

template <typename V>
hipError_t dispatch(const int32_t* ids, const int32_t* n_dev, int64_t n_cap, const void* feats,
                    int64_t num_nodes, int64_t row_bytes, void* out, uint32_t* status, hipStream_t s) {
  constexpr int U = 4;
  const int64_t cpr = (row_bytes + sizeof(V) - 1) / sizeof(V);
  int G = 64;
  if (cpr <= 4) G = 4;
  else if (cpr <= 8) G = 8;
  else if (cpr <= 16) G = 16;
  else if (cpr <= 32) G = 32;
  const int64_t rows_per_block = (256 / G) * U;
  int64_t blocks = (n_cap + rows_per_block - 1) / rows_per_block;
  if (blocks > GMB_GATHER_MAX_BLOCKS) blocks = GMB_GATHER_MAX_BLOCKS;
  if (blocks < 1) blocks = 1;
  const dim3 grid(static_cast<unsigned>(blocks)), block(256);
  const char* f = static_cast<const char*>(feats);
  char* o = static_cast<char*>(out);
#define GMB_GATHER(GG)                                                                                        \
  if (row_bytes % static_cast<int64_t>(sizeof(V)) == 0)                                                       \
    hipLaunchKernelGGL((k_gather<V, GG, U, true>), grid, block, 0, s, ids, n_dev, n_cap, f, num_nodes,        \
                       row_bytes, o, status);                                                                 \
  else                                                                                                        \
    hipLaunchKernelGGL((k_gather<V, GG, U, false>), grid, block, 0, s, ids, n_dev, n_cap, f, num_nodes,       \
                       row_bytes, o, status)
  switch (G) {
    case 4: GMB_GATHER(4); break;
    case 8: GMB_GATHER(8); break;
    case 16: GMB_GATHER(16); break;
    case 32: GMB_GATHER(32); break;
    default: GMB_GATHER(64); break;
  }
#undef GMB_GATHER
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gather(const int32_t* ids, const int32_t* n_dev, int64_t n_cap, const void* feats,
                         int64_t num_nodes, int64_t row_bytes, void* out, uint32_t* status,
                         hipStream_t s) {
  if (row_bytes >= 16) return dispatch<uint4>(ids, n_dev, n_cap, feats, num_nodes, row_bytes, out, status, s);
  if (row_bytes >= 8) return dispatch<uint2>(ids, n_dev, n_cap, feats, num_nodes, row_bytes, out, status, s);
  if (row_bytes >= 4) return dispatch<uint32_t>(ids, n_dev, n_cap, feats, num_nodes, row_bytes, out, status, s);
  return dispatch<uint16_t>(ids, n_dev, n_cap, feats, num_nodes, row_bytes, out, status, s);
}

}  // namespace gmb
