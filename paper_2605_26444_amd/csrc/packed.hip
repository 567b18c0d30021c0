// The paper's own system design as a component (Sec. 3.3 "Avoiding sparse computation via asynchronous
// gathering"; the weight-gather row of Table 4; the repacked-weights row of Table 6): a pre-allocated packed
// buffer holds one copy of every active row; after a vocabulary update only the rows of ids that entered the
// active set are copied in -- on a stream of the caller's choice, so that the copy hides behind the draft
// backbone -- and the head is a dense product on the packed buffer.
//
// Slots are stable: an id keeps its slot while it stays active, a leaving id frees its slot, an entering id
// takes the lowest free one.  Slot order is therefore not id order; the head kernels write the logits of the row
// in slot s to the column out_pos[s] = position of that id in the ascending active list, so logits come out in
// exactly the layout of nanospec_sparse_head and the selection (ties by lower id) applies unchanged.
#include "common.h"

namespace nanospec {

constexpr int kSyncThreads = 1024;

// exclusive rank of `pred` among the workgroup's threads in thread order, and the workgroup total; sc: 17 ints of LDS
__device__ __forceinline__ int block_rank(bool pred, int* sc, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long bal = __ballot(pred);
  const int before = __popcll(bal & ((1ull << lane) - 1ull));
  __syncthreads();                                   // sc may still be read from the previous call
  if (lane == 0) sc[wave] = __popcll(bal);
  __syncthreads();
  int off = 0, tot = 0;
  for (int w = 0; w < kSyncThreads / 64; ++w) {
    const int t = sc[w];
    off += w < wave ? t : 0;
    tot += t;
  }
  *total = tot;
  return off + before;
}

// One workgroup: bring slot tables in line with the active list of sequence 0.
//   1. every slot whose id is no longer active (window bitmap | T bitmap) is freed;
//   2. the free slots are listed in ascending order;
//   3. every active id without a slot takes the next free one and goes on the copy list;
//   4. out_pos[slot] = position of the slot's id in the ascending list; hi = slots that may hold a row.
__global__ __launch_bounds__(kSyncThreads) void packed_sync_kernel(VocabPtrs p, PackedPtrs k) {
  __shared__ int sc[32];
  const int tid = threadIdx.x;
  const int n = p.n[0], cap = k.cap;
  int nfree = 0;
  for (int s0 = 0; s0 < cap; s0 += kSyncThreads) {
    const int s = s0 + tid;
    bool isfree = false;
    if (s < cap) {
      const int id = k.slot_id[s];
      isfree = id < 0;
      if (id >= 0) {
        const uint32_t bits = p.wbit[id >> 5] | p.tbit[id >> 5];
        if (!((bits >> (id & 31)) & 1u)) {
          k.slot_of[id] = -1;
          k.slot_id[s] = -1;
          k.out_pos[s] = -1;
          isfree = true;
        }
      }
    }
    int tot;
    const int r = block_rank(isfree, sc, &tot);
    if (isfree) k.free_list[nfree + r] = s;
    nfree += tot;
  }
  __syncthreads();                                   // free_list and slot_of are complete (one workgroup, one L1)
  int ncopy = 0, top = -1;
  for (int j0 = 0; j0 < n; j0 += kSyncThreads) {
    const int j = j0 + tid;
    int id = -1, sl = -1;
    if (j < n) {
      id = p.ids[j];
      sl = k.slot_of[id];
    }
    const bool fresh = j < n && sl < 0;
    int tot;
    const int r = block_rank(fresh, sc, &tot);
    if (fresh) {
      sl = k.free_list[ncopy + r];                   // n <= cap and every active id holds one slot: there is one
      k.slot_of[id] = sl;
      k.slot_id[sl] = id;
      k.copy_list[2 * (ncopy + r)] = id;
      k.copy_list[2 * (ncopy + r) + 1] = sl;
    }
    if (j < n) k.out_pos[sl] = j;
    top = max(top, sl);
    ncopy += tot;
  }
  // highest slot in use
  for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o));
  __syncthreads();
  if ((tid & 63) == 0) sc[tid >> 6] = top;
  __syncthreads();
  if (tid == 0) {
    int t = -1;
    for (int w = 0; w < kSyncThreads / 64; ++w) t = max(t, sc[w]);
    k.scal[0] = t + 1;                               // hi
    k.scal[1] = ncopy;
  }
}

// The same for capacities of up to Q x 4096 slots in two memory round trips and one scan (the walk above takes two round
// trips, two ranks and their stores' latency per 1024 slots and again per 1024 ids: 8.4 us at 3750 slots).  Thread t holds slots and list
// positions q * 4096 + 4t .. + 3: slot ids and listed ids are asked for together, then the bitmap words of the former
// and the slots of the latter -- a listed id's slot is not freed by this call, so the two do not wait for each other.
// Free slots and ids without a slot are ranked in one scan; the free list lives in LDS.  All stores come last: the
// f-th free slot is taken by the f-th new id, so the thread that frees a slot clears its tables only if it stays free.
template <int Q>
__global__ __launch_bounds__(kSyncThreads) void packed_sync_short_kernel(VocabPtrs p, PackedPtrs k) {
  constexpr int NW = kSyncThreads / 64;
  __shared__ int s_free[Q * 4096];
  __shared__ int2 s_tot[Q][NW];
  __shared__ int s_top;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cap = k.cap;                                   // a multiple of 64, as are the lists' lengths
  int sid[Q][4], id[Q][4], sl[Q][4];
  uint32_t fr[Q], nw[Q];                                   // bit e: slot free (bit 4 + e: by this call) / id without a slot
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int s = q * 4096 + tid * 4;
    const int4 a = *reinterpret_cast<const int4*>(k.slot_id + (s < cap ? s : 0));
    const int4 b = *reinterpret_cast<const int4*>(p.ids + (s < cap ? s : 0));
    sid[q][0] = a.x; sid[q][1] = a.y; sid[q][2] = a.z; sid[q][3] = a.w;
    id[q][0] = b.x; id[q][1] = b.y; id[q][2] = b.z; id[q][3] = b.w;
  }
  const int n = p.n[0];
  if (tid == 0) s_top = -1;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int s = q * 4096 + tid * 4;
    uint32_t word[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int w = sid[q][e] >= 0 ? sid[q][e] >> 5 : 0;
      word[e] = p.wbit[w] | p.tbit[w];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) sl[q][e] = k.slot_of[s + e < n ? id[q][e] : 0];   // entries past n may be anything
    fr[q] = nw[q] = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool gone = sid[q][e] >= 0 && !((word[e] >> (sid[q][e] & 31)) & 1u);
      if (s < cap && (sid[q][e] < 0 || gone)) fr[q] |= (gone ? 17u : 1u) << e;
      if (s + e < n && sl[q][e] < 0) nw[q] |= 1u << e;
    }
  }
  // ranks in (q, thread, e) order = ascending slots / ids
  int2 incl[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    incl[q] = make_int2(__popc(fr[q] & 15u), __popc(nw[q]));
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int x = __shfl_up(incl[q].x, o), y = __shfl_up(incl[q].y, o);
      incl[q].x += lane >= o ? x : 0;
      incl[q].y += lane >= o ? y : 0;
    }
    if (lane == 63) s_tot[q][wave] = incl[q];
  }
  __syncthreads();
  int fbase[Q], nbase[Q], ftot = 0, ncopy = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    int fo = ftot, no = ncopy;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int2 t = s_tot[q][w];
      fo += w < wave ? t.x : 0;
      no += w < wave ? t.y : 0;
      ftot += t.x;
      ncopy += t.y;
    }
    fbase[q] = fo + incl[q].x - __popc(fr[q] & 15u);
    nbase[q] = no + incl[q].y - __popc(nw[q]);
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    int f = fbase[q];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if ((fr[q] >> e) & 1u) s_free[f++] = q * 4096 + tid * 4 + e;
  }
  __syncthreads();
  int top = -1;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    int r = nbase[q];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if ((nw[q] >> e) & 1u) sl[q][e] = s_free[r++];       // n <= cap and every active id holds one slot: there is one
      if (q * 4096 + tid * 4 + e < n) top = max(top, sl[q][e]);
    }
  }
  for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o));
  if (lane == 0) atomicMax(&s_top, top);
  __syncthreads();
  if (tid == 0) {
    k.scal[0] = s_top + 1;                                 // hi
    k.scal[1] = ncopy;
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    int f = fbase[q], r = nbase[q];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int s = q * 4096 + tid * 4 + e;                // slot and list position
      if ((fr[q] >> (4 + e)) & 1u) {
        k.slot_of[sid[q][e]] = -1;
        if (f >= ncopy) {
          k.slot_id[s] = -1;
          k.out_pos[s] = -1;
        }
      }
      f += (fr[q] >> e) & 1u;
      if (s < n) k.out_pos[sl[q][e]] = s;
      if ((nw[q] >> e) & 1u) {
        k.slot_of[id[q][e]] = sl[q][e];
        k.slot_id[sl[q][e]] = id[q][e];
        k.copy_list[2 * r] = id[q][e];
        k.copy_list[2 * r + 1] = sl[q][e];
        ++r;
      }
    }
  }
}

// Copy the listed rows W[id] -> buf[slot]: the weight-gather kernel.  Two small workgroups per compute unit (a decoding step copies a
// row or two, and then the launch is all there is: a request of 16 steps 365 us with 256 workgroups of 1024 threads, 359 with 512 of
// 256, 364 with 256 of 256), four 16-byte pieces per thread in flight for the first gather.
__global__ __launch_bounds__(256) void packed_copy_kernel(const uint4* __restrict__ W, PackedPtrs k, int row_vec /* 16-byte pieces per row */) {
  const int ncopy = k.scal[1];
  uint4* buf = reinterpret_cast<uint4*>(k.buf);
  const int64_t total = (int64_t)ncopy * row_vec, stride = (int64_t)gridDim.x * 256;
  for (int64_t t0 = (int64_t)blockIdx.x * 256 + threadIdx.x; t0 < total; t0 += 4 * stride) {
    uint4 v[4];
    int64_t to[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t t = t0 + u * stride;
      const uint32_t tc = (uint32_t)(t < total ? t : t0);   // below 2^32: capacity * d / 8
      const uint32_t e = tc / (uint32_t)row_vec, i = tc % (uint32_t)row_vec;
      const int2 cs = *reinterpret_cast<const int2*>(k.copy_list + 2 * (int64_t)e);
      v[u] = W[(int64_t)cs.x * row_vec + i];
      to[u] = (int64_t)cs.y * row_vec + i;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (t0 + u * stride < total) buf[to[u]] = v[u];
  }
}

__global__ __launch_bounds__(256) void packed_reset_kernel(PackedPtrs k, int V) {
  const int i = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
  for (int v = i; v < V; v += stride) k.slot_of[v] = -1;
  for (int s = i; s < k.cap; s += stride) {
    k.slot_id[s] = -1;
    k.out_pos[s] = -1;
  }
  if (i == 0) {
    k.scal[0] = 0;
    k.scal[1] = 0;
  }
}

hipError_t launch_packed_reset(const nanospec_state* st, hipStream_t s) {
  packed_reset_kernel<<<256, 256, 0, s>>>(st->pk, st->V);
  return hipGetLastError();
}

hipError_t launch_packed_gather(const nanospec_state* st, const void* W, hipStream_t s) {
  const int cap = st->pk.cap;
  if (cap <= 4096) packed_sync_short_kernel<1><<<1, kSyncThreads, 0, s>>>(st->vp, st->pk);
  else if (cap <= 8192) packed_sync_short_kernel<2><<<1, kSyncThreads, 0, s>>>(st->vp, st->pk);
  else packed_sync_kernel<<<1, kSyncThreads, 0, s>>>(st->vp, st->pk);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  packed_copy_kernel<<<512, 256, 0, s>>>(static_cast<const uint4*>(W), st->pk, st->d / 8);
  return hipGetLastError();
}

}  // namespace nanospec
