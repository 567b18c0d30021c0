// Internal declarations shared by the translation units of libnanospec (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "choose.h"
#include "nanospec.h"

namespace nanospec {

constexpr int kVocabThreads = 1024;   // one workgroup per sequence in the vocabulary kernel
constexpr int kTopkThreads = 1024;    // single-pass top-k workgroup
constexpr int kMaxK = 64;
constexpr int kCandMax = 256;          // top-k fast path: most candidates ranked directly

// Sums over lanes of integers by DPP (row of 16 lanes; a lane without a source adds 0): an instruction per step where a shuffle through LDS is several.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_add_int(int x) {
  return x + __builtin_amdgcn_update_dpp(0, x, CTRL, ROW_MASK, 0xf, false);
}

// inclusive prefix sum over the 64 lanes: Hillis-Steele inside each row of 16 (row_shr 1, 2, 4, 8), then the row totals
// carried across (row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3)
__device__ __forceinline__ int wave_incl_scan(int x) {
  x = dpp_add_int<0x111, 0xf>(x);
  x = dpp_add_int<0x112, 0xf>(x);
  x = dpp_add_int<0x114, 0xf>(x);
  x = dpp_add_int<0x118, 0xf>(x);
  x = dpp_add_int<0x142, 0xa>(x);
  return dpp_add_int<0x143, 0xc>(x);
}

// sum over each row of 16 lanes, in all of them (quad_perm neighbours, row_half_mirror, row_mirror)
__device__ __forceinline__ int row_sum(int x) {
  x = dpp_add_int<0xB1, 0xf>(x);
  x = dpp_add_int<0x4E, 0xf>(x);
  x = dpp_add_int<0x141, 0xf>(x);
  return dpp_add_int<0x140, 0xf>(x);
}

// The clobber of M0 is what it says: the compiler keeps nothing there across statements (it writes M0 in front of each use of its
// own), and warns at every inlined copy only because it reserves the register.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_fetch16(uint32_t lds, const void* base, uint32_t off) {
  // 16 bytes per lane from base + off straight into LDS at lds + 16 * lane; no destination register.  A load into LDS may read M0
  // one wait state after a scalar write of it, and nothing puts that state between two instructions of one statement: the s_nop.
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop

// Per-sequence offsets travel by value in the kernel argument block (no H2D copy, graph-safe).
struct Offsets {
  int32_t v[NANOSPEC_MAX_BATCH + 1];
};

struct VocabPtrs {
  int32_t* ring;        // [batch][window]
  uint32_t* cnt;        // [batch][V]
  uint32_t* wbit;       // [batch][nwords]
  uint32_t* tbit;       // [batch][nwords]
  int32_t* ids;         // [batch][cap]
  int32_t* n;           // [batch]
  int32_t* pos;         // [batch] next ring slot
  int32_t* fill;        // [batch] valid ring entries
  int32_t* err;         // [1] sticky flags
  int32_t V, window, nwords, cap;
};

// Packed-buffer variant (one sequence): slot tables and the row copies.
struct PackedPtrs {
  uint16_t* buf;        // [cap][d] bf16: one row per slot
  int32_t* slot_of;     // [V]   slot that holds the id's row, or -1: of packed_sync_kernel, which takes what does not fit packed_sync_short_kernel
  int32_t* slot_id;     // [cap] id whose row the slot holds, or -1
  int32_t* out_pos;     // [cap] position of that id in the ascending active list, or -1
  int32_t* free_list;   // [cap] scratch of one gather: free slots ascending, of the same kernel
  int32_t* copy_list;   // [cap][2] scratch of one gather: (id, slot) of the rows to copy
  int32_t* scal;        // [0] slots that may hold a row (highest slot in use + 1), [1] rows on the copy list
  int32_t cap;
};

// Batch-union head (several sequences): rows shared by many sequences, and what is left per sequence.
struct UnionPtrs {
  uint32_t* shared_bits;  // [nwords] bit = id held by at least min_share sequences
  int32_t* shared_ids;    // [shared_cap] the lowest shared_cap such ids, ascending
  int32_t* shared_n;      // [groups] their number, repeated once per group of 64 hidden rows
  int32_t* shared_pos;    // [batch][shared_cap] column of shared row r in the sequence's logits, -1 if the sequence lacks it
  int32_t* rest_ids;      // [batch][cap] the sequence's other active ids, ascending
  int32_t* rest_pos;      // [batch][cap] their columns
  int32_t* rest_n;        // [batch]
  // What the head works from where the overlap decides (union_feeds in choose.h), else null: the lists above, or nothing shared and every list whole.
  int2* parts;            // [workgroups of the count] pairs of a sequence and an active id / those of ids that qualify as shared (the lists count those with room)
  int32_t* head_ids;      // [batch][cap]
  int32_t* head_pos;      // [batch][cap]
  int32_t* head_n;        // [batch]
  int32_t* head_shared_n; // [groups] as shared_n, or 0
  int32_t shared_cap, min_share;
};

}  // namespace nanospec

struct nanospec_state {
  int32_t V, d, batch, window, topk_cap, m_cap, k_cap;
  int32_t device;
  nanospec_layout layout;
  nanospec::VocabPtrs vp;
  char* base;               // the one device allocation everything lives in
  float* partial;           // split-K partial logits
  char* topk_ws;            // two-pass top-k candidates (lists longer than 16 384, where they are selected in chunks)
  int64_t partial_bytes, topk_ws_bytes;
  int32_t* h_err_pinned;    // pinned host word for reading the device flags
  int vocab_lds_bytes, unique_lds_bytes, unique_cap, fifo_lds_bytes;
  int32_t policy, policy_next;   // vocabulary reading in force / chosen for the next init
  nanospec::PackedPtrs pk;       // packed-buffer variant; pk.buf == nullptr until nanospec_packed_enable
  char* pk_base;                 // its one device allocation
  nanospec::UnionPtrs un;        // batch-union head; un_base == nullptr until nanospec_union_enable
  char* un_base;
  int32_t un_groups;             // groups of 64 hidden rows at M = m_cap
};

namespace nanospec {

// vocab.hip
hipError_t launch_vocab_clear(const nanospec_state* st, hipStream_t s);
hipError_t launch_vocab_init(const nanospec_state* st, const int32_t* d_ctx, const Offsets& coff, const int32_t* d_topk,
                             const Offsets& toff, hipStream_t s);
hipError_t launch_vocab_apply(const nanospec_state* st, const int32_t* d_new, const Offsets& noff,
                              const int32_t* d_topk, const Offsets& toff, int replace_T, hipStream_t s);
hipError_t vocab_configure(nanospec_state* st);
hipError_t vocab_configure_device();
hipError_t launch_vocab_append_unique(const nanospec_state* st, const int32_t* d_cand, int per_seq, int64_t stride,
                                      hipStream_t s);

// head.hip
hipError_t head_configure_device();
// logits[b][m][j] for j < n_b (n read on the device).  ids == nullptr: identity list of n_fixed rows.
// opos != nullptr (row stride ids_stride): row j's logits go to column opos[j] instead, nowhere if negative.
hipError_t launch_head(const void* W, const void* H, const int32_t* ids, const int32_t* n_dev, int32_t n_fixed,
                       int32_t cap_rows, int32_t V, int32_t batch, int32_t M, int32_t d, int64_t ld_logits,
                       int64_t ids_stride, float* logits, float* partial, int64_t partial_bytes, const int32_t* opos,
                       hipStream_t s);

// every row of one list against rows_total hidden rows of several sequences (seq_rows each); columns per sequence
hipError_t launch_head_shared(const void* W, const void* H, const int32_t* ids, const int32_t* n_rep, int32_t cap_rows, int32_t V,
                              int32_t rows_total, int32_t seq_rows, int32_t d, int64_t ld_logits, float* logits, const int32_t* opos,
                              int64_t opos_stride, hipStream_t s);

// wide.hip: register-blocked product
hipError_t launch_head_wide_shared(const void* W, const void* H, const int32_t* ids, const int32_t* n_dev, int32_t cap_rows, int32_t V,
                                   int32_t rows_total, int32_t seq_rows, int32_t d, int64_t ld, float* logits, const int32_t* opos,
                                   int64_t opos_stride, hipStream_t s);
hipError_t wide_configure_device();
hipError_t launch_head_wide(const void* W, const void* H, const int32_t* ids, const int32_t* n_dev, int32_t n_fixed, int32_t cap_rows,
                            int32_t V, int32_t batch, int32_t M, int32_t d, int64_t ld, int64_t ids_stride, float* logits,
                            const int32_t* opos, hipStream_t s);

// hold.hip: up to 16 hidden rows held in registers
hipError_t hold_configure_device();
hipError_t launch_head_hold(const void* W, const void* H, const int32_t* ids, const int32_t* n_dev, int32_t n_fixed, int32_t V, int32_t batch, int32_t M,
                            int32_t d, int64_t ld, int64_t ids_stride, float* logits, const int32_t* opos, hipStream_t s);

// kslice.hip: 17 to 64 hidden rows, K sliced over the wavefronts
hipError_t kslice_configure_device();
hipError_t launch_head_kslice(const void* W, const void* H, const int32_t* ids, const int32_t* n_dev, int32_t cap_rows, int32_t V, int32_t batch, int32_t M,
                              int32_t d, int64_t ld, int64_t ids_stride, float* logits, const int32_t* opos, hipStream_t s);

// union.hip
hipError_t union_configure_device();
hipError_t launch_union_reset(const nanospec_state* st, hipStream_t s);
hipError_t launch_union_build(const nanospec_state* st, hipStream_t s);

// topk.hip
int64_t topk_workspace_bytes(int32_t cap, int32_t rows, int32_t k);
hipError_t launch_topk(const float* logits, int64_t ld, const int32_t* ids, int64_t ids_stride, const int32_t* n_dev,
                       int32_t n_fixed, int32_t cap, int64_t expected /* see topk_expected */, int32_t batch, int32_t M, int32_t k,
                       int32_t* out_ids, float* out_vals, bool logprob, char* ws, int64_t ws_bytes, hipStream_t s);

// packed.hip
hipError_t packed_configure_device();
hipError_t launch_packed_reset(const nanospec_state* st, hipStream_t s);
hipError_t launch_packed_gather(const nanospec_state* st, const void* W, hipStream_t s);

// calib.hip
hipError_t launch_calib_stream(const void* buf, int64_t bytes, void* sink, hipStream_t s);
hipError_t launch_calib_valu_head(const void* W, const void* H, int32_t V, int32_t d, int32_t M, const int32_t* ids,
                                  const int32_t* n_dev, int32_t cap, float* logits, hipStream_t s);
hipError_t calib_configure_device();
hipError_t launch_calib_gather(const void* W, int32_t V, int32_t d, const int32_t* ids, const int32_t* n_dev, int32_t cap,
                               void* sink, hipStream_t s);

}  // namespace nanospec
