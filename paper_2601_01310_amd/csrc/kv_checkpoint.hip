// Incremental KV-segment checkpoint and request-level restoration (§6.1,
// §6.2), with host memory in the role of the checkpoint store.
//
// Two ways to copy: a kernel over an arbitrary list of segments, on a
// bounded number of workgroups; and, for segments at a constant stride (one
// decode step of a [layer][request][position] region), one strided copy on
// the copy engine, which leaves the compute units to the forward.
//
// The KV region and the store have the same layout, so a segment's offset
// in the region is its offset in the store. A checkpoint call copies a batch
// of segments (one block per segment at a time, 16-byte loads and stores
// straight into host-visible memory), writes one log record per segment,
// makes its writes visible system-wide, and then, in a second kernel that
// starts only after every copy has finished, publishes the commit record:
// the sequence number after the batch's last, so every number below it has
// landed. Restoration reads the commit record and copies back only the
// segments numbered below it.
#include "tg.h"
#include "tg_device.h"
#include "tg_launch.h"

namespace tg {
namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ bool seg_ok(uint64_t off, uint64_t bytes, uint64_t limit) {
  return (off % 16 == 0) && (bytes % 16 == 0) && off <= limit && bytes <= limit - off;
}

// One wave per SIMD and few registers: beside a forward a block of it shares
// its CU with a block of the grouped GEMM, which leaves 24 registers per lane.
// (16 waves per block, four segments at a time, copy 4096 segments of 4 KB in
// 328 us instead of 364, but then the GEMM's block waits for the whole copy:
// a decode forward beside it takes 757 us instead of 561.)
__global__ __launch_bounds__(kBlock) void ckpt_copy_kernel(
    const uint4* __restrict__ kv, uint64_t kv_bytes, const uint64_t* __restrict__ seg_off,
    const uint32_t* __restrict__ seg_bytes, int n, uint64_t first_seq, uint4* store,
    tg_ckpt_record* log, int log_cap) {
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    const uint64_t o = seg_off[i];
    const uint32_t b = seg_bytes[i];
    const bool ok = seg_ok(o, b, kv_bytes);
    if (ok) {
      const uint64_t base = o / 16;
      for (uint32_t c = threadIdx.x; c < b / 16; c += kBlock) store[base + c] = kv[base + c];
    }
    // The log is a ring of log_cap records: of a batch longer than the ring
    // only the last log_cap records are kept, so no two writes collide.
    if (threadIdx.x == 0 && i >= n - log_cap) {
      tg_ckpt_record r;
      r.seq = first_seq + (uint64_t)i;
      r.offset = o;
      r.bytes = ok ? b : 0;  // 0: rejected (misaligned or outside the region)
      log[r.seq % (uint64_t)log_cap] = r;
    }
  }
  __threadfence_system();
}

__global__ void ckpt_commit_kernel(uint64_t* commit, uint64_t seq) {
  __threadfence_system();
  __hip_atomic_store(commit, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Records of a strided batch (segment i at first_offset + i * pitch), then,
// after every record, the commit record; one block.
__global__ __launch_bounds__(kBlock) void ckpt_log_commit_kernel(
    uint64_t first_offset, uint64_t pitch, uint32_t seg_bytes, int n, uint64_t first_seq,
    tg_ckpt_record* log, int log_cap, uint64_t* commit) {
  for (int i = max(0, n - log_cap) + threadIdx.x; i < n; i += kBlock) {
    tg_ckpt_record r;
    r.seq = first_seq + (uint64_t)i;
    r.offset = first_offset + (uint64_t)i * pitch;
    r.bytes = seg_bytes;
    log[r.seq % (uint64_t)log_cap] = r;
  }
  __threadfence_system();
  __syncthreads();
  if (commit && threadIdx.x == 0)
    __hip_atomic_store(commit, first_seq + (uint64_t)n, __ATOMIC_RELEASE,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// Restore: status of segment i, with the commit record as it was read.
__device__ __forceinline__ uint8_t restore_status(uint64_t committed, uint64_t seq, uint64_t src,
                                                  uint64_t dst, uint32_t b, uint64_t store_bytes,
                                                  uint64_t kv_bytes) {
  if (!seg_ok(src, b, store_bytes) || !seg_ok(dst, b, kv_bytes)) return 2;
  return seq < committed ? 1 : 0;  // not committed: its bytes may be incomplete
}

__device__ __forceinline__ uint64_t read_commit(const uint64_t* commit) {
  return __hip_atomic_load(commit, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// STATUS: the kernel reads the commit record and writes the status itself;
// otherwise kv_restore_status_kernel ran before it.
template <bool STATUS>
__global__ __launch_bounds__(kBlock) void kv_restore_kernel(
    const uint4* store, uint64_t store_bytes, const uint64_t* commit,
    const uint64_t* __restrict__ seq, const uint64_t* __restrict__ src,
    const uint64_t* __restrict__ dst, const uint32_t* __restrict__ bytes, int n,
    uint4* __restrict__ kv, uint64_t kv_bytes, uint8_t* status) {
  uint64_t committed = 0;
  if (STATUS) committed = read_commit(commit);
  else __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");  // the store's bytes, from where they are
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    const uint32_t b = bytes[i];
    const uint64_t s0 = src[i], d0 = dst[i];
    const uint8_t st =
        STATUS ? restore_status(committed, seq[i], s0, d0, b, store_bytes, kv_bytes) : status[i];
    if (st == 1)
      for (uint32_t c = threadIdx.x; c < b / 16; c += kBlock) kv[d0 / 16 + c] = store[s0 / 16 + c];
    if (STATUS && threadIdx.x == 0) status[i] = st;
  }
}

__global__ __launch_bounds__(kBlock) void kv_restore_status_kernel(
    uint64_t store_bytes, const uint64_t* commit, const uint64_t* __restrict__ seq,
    const uint64_t* __restrict__ src, const uint64_t* __restrict__ dst,
    const uint32_t* __restrict__ bytes, int n, uint64_t kv_bytes, uint8_t* __restrict__ status) {
  __shared__ uint64_t committed;
  if (threadIdx.x == 0) committed = read_commit(commit);
  __syncthreads();
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock)
    status[i] =
        restore_status(committed, seq[i], src[i], dst[i], bytes[i], store_bytes, kv_bytes);
}

// A restore of more than kRestoreAlone segments reads the commit record in a
// kernel of its own, and kRestoreBlocks blocks copy. The record lies across the
// host's link, where each block's read of it costs about 0.37 us, one after
// the other, so a copy whose blocks all read it pays for every block. us, all
// reading it with 4096 blocks, with 48, and this way with 256:
//   host memory    200 x    4 KB      107    36    29
//                 4096 x    4 KB     1965   314   310   (the link's rate)
//   device memory  200 x    4 KB       76    22    12
//                 4096 x    4 KB     1212    59    24
//                 1000 x 1024 KB      796  2532   702
// 512 blocks copy the last in 445, but the 4096 segments from the host in 326.
// Up to a dozen segments the second launch is the dearer: 8 take 7 us in one
// kernel and 9 in two, 16 10 and 9.
constexpr int kRestoreBlocks = 256;
constexpr int kRestoreAlone = 12;

int grid_for(int n, int max_blocks) { return n < max_blocks ? n : max_blocks; }

}  // namespace

hipError_t launch_kv_checkpoint(const void* kv, size_t kv_bytes, const uint64_t* seg_off,
                                const uint32_t* seg_bytes, int n, uint64_t first_seq, void* store,
                                tg_ckpt_record* log, int log_cap, uint64_t* commit, int max_blocks,
                                hipStream_t stream) {
  if (n > 0)
    hipLaunchKernelGGL(ckpt_copy_kernel, dim3(grid_for(n, max_blocks)), dim3(kBlock), 0, stream,
                       static_cast<const uint4*>(kv), (uint64_t)kv_bytes, seg_off, seg_bytes, n,
                       first_seq, static_cast<uint4*>(store), log, log_cap);
  if (commit && n > 0)
    hipLaunchKernelGGL(ckpt_commit_kernel, dim3(1), dim3(1), 0, stream, commit,
                       first_seq + (uint64_t)n);
  return hipGetLastError();
}

hipError_t launch_kv_checkpoint_strided(const void* kv, uint64_t first_offset, uint64_t pitch,
                                        uint32_t seg_bytes, int n, uint64_t first_seq,
                                        void* store, tg_ckpt_record* log, int log_cap,
                                        uint64_t* commit, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  // One strided copy by the copy engine: no compute unit is used. The store
  // has the region's layout, so source and destination share the pitch.
  hipError_t e = hipMemcpy2DAsync(static_cast<char*>(store) + first_offset, pitch,
                                  static_cast<const char*>(kv) + first_offset, pitch, seg_bytes, n,
                                  hipMemcpyDefault, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(ckpt_log_commit_kernel, dim3(1), dim3(kBlock), 0, stream, first_offset, pitch,
                     seg_bytes, n, first_seq, log, log_cap, commit);
  return hipGetLastError();
}

hipError_t launch_kv_restore(const void* store, size_t store_bytes, const uint64_t* commit,
                             const uint64_t* seq, const uint64_t* src, const uint64_t* dst,
                             const uint32_t* bytes, int n, void* kv, size_t kv_bytes,
                             uint8_t* status, hipStream_t stream) {
  if (n <= 0) return hipGetLastError();
  const dim3 grid(grid_for(n, kRestoreBlocks)), block(kBlock);
  const uint4* const from = static_cast<const uint4*>(store);
  uint4* const to = static_cast<uint4*>(kv);
  if (n <= kRestoreAlone) {
    hipLaunchKernelGGL(kv_restore_kernel<true>, grid, block, 0, stream, from, (uint64_t)store_bytes,
                       commit, seq, src, dst, bytes, n, to, (uint64_t)kv_bytes, status);
  } else {
    hipLaunchKernelGGL(kv_restore_status_kernel, dim3(grid_for((n + kBlock - 1) / kBlock, 16)),
                       block, 0, stream, (uint64_t)store_bytes, commit, seq, src, dst, bytes, n,
                       (uint64_t)kv_bytes, status);
    hipLaunchKernelGGL(kv_restore_kernel<false>, grid, block, 0, stream, from,
                       (uint64_t)store_bytes, commit, seq, src, dst, bytes, n, to,
                       (uint64_t)kv_bytes, status);
  }
  return hipGetLastError();
}

}  // namespace tg
