// The "clean views" stage in toy form (Section 3 of the paper, "Clean views": null values are
// filled, fields are taken out of a JSON-like column, instances are dropped by a custom filter;
// Section 4 puts the stage on the GPU next to feature extraction).  The paper gives no algorithm
// for any of the three; the contract built here is the one stated at fbx_clean_create in
// include/fbx.h.  Output is a cleaned text buffer plus record offsets, in input order, ready to be
// handed to fbx_extract without leaving the device.
//
// A cleaned record is its text with a few fields replaced: most bytes only move.  Two launches over
// tiles of T consecutive records.  The first one measures: a workgroup copies a tile's text into LDS
// with 16-byte loads that all its lanes share, groups of lanes split each record at its tabs into a
// table of field ends (split_bytes, the extraction path's splitter), lanes that are (record, field)
// pairs apply the operators, to the fields that have any, and what they change is left in the scratch
// buffer as a list of segments: where in the tile's output a run of bytes starts, and where in LDS it
// comes from (the text, or the operators' arguments behind it).  The second one writes: it stages the
// text of the kept records at the same places, and its lanes are 16-byte chunks of the output.  A
// tile's place in the output is the sum over the tiles before it: a workgroup takes a run of consecutive
// tiles in both launches and leaves the run's sum, so that one sum over the runs before its own is all
// it takes.  (Nothing is handed out by counters: atomic adds of one address from the whole chip pass
// at about 75 a microsecond, and a tile takes less than that.)
// A tile whose text does not fit the section is read in place, a record per thread; so is everything
// when a specification has too many fields for the tables.  Where there is no room for segments (in the
// scratch buffer, or in LDS beside many operators) both launches of k_clean_tile apply the operators.
//
// (One launch with a look-back between tiles instead was built and is slower, 0.71 ms for the batch
// at k_clean_measure_tile: a tile waits for all the tiles that were started before it, some of a
// thousand in flight are always late, and no work is left to do meanwhile.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "fbx_device.h"
#include "fbx_split.h"

using namespace fbx;

namespace {

enum CleanKind : uint32_t { CK_FILL = 1, CK_KEY = 2, CK_KEEP = 3, CK_NONE = 4 };  // (CK_NONE: a key that no pair can have)

struct CleanOp {
  uint32_t kind, field, arg_off, arg_len;
};

struct OpField {
  uint32_t field, first_op;  // its operators are ops[first_op .. the next entry's first_op)
  uint32_t keyed;            // the first of them looks a key up
};

struct CleanParams {
  const uint8_t* raw;
  uint64_t raw_len;
  const uint64_t* rec_off;
  uint64_t n_records;
  const CleanOp* ops;         // sorted by field, spec order inside a field
  const uint32_t* first_op;   // [n_fields + 1] the operators of field k are ops[first_op[k] .. first_op[k + 1])
  const uint8_t* args;
  uint32_t n_fields;
  uint32_t n_of, n_ops, args_bytes, n_keyed;
  const uint32_t* keyed;      // [n_keyed] entries of `of` whose first operator looks a key up
  const OpField* of;          // [n_of + 1] the fields that have operators, in order
  uint32_t* lens;             // (kernels without segments) [2][n_records]: bytes of the cleaned record (0: dropped); 1 if kept
  const uint64_t* base;       // [2][n_records]: where a kept record goes; its number among the kept ones
  const uint64_t* total;      // [2]: bytes of the output; kept records
  uint8_t* out;
  uint64_t out_cap;
  uint64_t* out_off;
  Ctrl* ctrl;
  // the tile kernels: what the measuring launch leaves for the writing one
  uint64_t* rec_out;    // [n_records] where the record starts in its tile's output; kDropped
  uint64_t* sums;       // [n_tiles] bytes of the tile's output
  uint64_t* run_sums;   // [2][gridDim.x] bytes of the output of a workgroup's tiles; kept records
  uint32_t* n_segs;     // [n_tiles] segments of the tile; kInPlace
  uint32_t* segs;       // [n_records][2 n_of + 3], a tile's segments at its first record's place
  uint32_t n_tiles, run;  // tiles; how many in a row a workgroup takes
  uint32_t log2T;       // records per tile
  uint32_t raw_cap;     // bytes of the text section in LDS (a multiple of 16)
  uint32_t row_stride;  // 16-bit entries per record in the table of field ends
  uint32_t o_args, o_rows, o_new, o_of, o_ops, o_keyed;  // where the tables start in LDS
  uint32_t o_seg, o_later;                      // (the writing launch; the text and the arguments lie at the same places)
  uint32_t o_len, o_src;                        // (the kernel without segments; its rows lie at o_rows)
  uint64_t* export_to;  // host memory: control block and totals, written by the last workgroup to finish (null: none)
};
constexpr uint64_t kDropped = ~0ull;
constexpr uint32_t kInPlace = ~0u, kMaxRuns = 4096;

constexpr uint32_t kCleanWaves = 6;  // a SIMD: six workgroups of four wavefronts on a compute unit, what the LDS admits
constexpr uint32_t kCleanThreads = 256, kCleanRawPad = 16, kCleanMaxT = 64;
constexpr uint32_t kTabRun = 0xffffu;  // a segment's source: tabs, as many as it takes (fields that the record lacks)

struct Bytes {
  const uint8_t* p;
  uint32_t n;
};

// value of the first pair "key:value" of v (pairs separated by ';') whose key is exactly name
__device__ Bytes key_value(Bytes v, const uint8_t* name, uint32_t name_len) {
  uint32_t p = 0;
  for (;;) {
    uint32_t q = p;
    while (q < v.n && v.p[q] != ';') ++q;
    uint32_t c = p;
    while (c < q && v.p[c] != ':') ++c;
    if (c < q && c - p == name_len) {
      bool same = true;
      for (uint32_t i = 0; i < name_len && same; ++i) same = v.p[p + i] == name[i];
      if (same) return Bytes{v.p + c + 1u, q - c - 1u};
    }
    if (q >= v.n) return Bytes{v.p, 0u};
    p = q + 1u;
  }
}

// Walks the F fields of one record, applies each field's operators and hands every cleaned field
// to emit(field bytes); returns false as soon as a filter drops the record.
template <class Emit>
__device__ bool clean_record(const CleanParams& C, const uint8_t* rec, uint32_t rn, Emit&& emit) {
  uint32_t p = 0;
  for (uint32_t k = 0; k < C.n_fields; ++k) {
    uint32_t q = p;
    while (q < rn && rec[q] != '\t') ++q;
    Bytes v{rec + (p <= rn ? p : rn), p <= rn ? q - p : 0u};  // (a missing field is empty)
    p = q < rn ? q + 1u : rn + 1u;
    for (uint32_t o = C.first_op[k]; o < C.first_op[k + 1]; ++o) {
      const CleanOp op = C.ops[o];
      const uint8_t* arg = C.args + op.arg_off;
      if (op.kind == CK_FILL) {
        if (v.n == 0) v = Bytes{arg, op.arg_len};
      } else if (op.kind == CK_KEY) {
        v = key_value(v, arg, op.arg_len);
      } else if (op.kind == CK_NONE) {
        v.n = 0;
      } else {
        bool ok = v.n >= op.arg_len;
        for (uint32_t i = 0; i < op.arg_len && ok; ++i) ok = v.p[i] == arg[i];
        if (!ok) return false;
      }
    }
    emit(v);
  }
  return true;
}

// the record of this thread without its trailing newline, or false (and an error bit) for bad offsets
__device__ bool clean_frame(const CleanParams& C, uint64_t r, const uint8_t*& rec, uint32_t& rn) {
  const uint64_t a = C.rec_off[r], b = C.rec_off[r + 1];
  if (a > b || b > C.raw_len) { atomicOr(&C.ctrl->err, (uint32_t)CE_OFFSETS); return false; }
  if (b - a >= (1ull << 31)) { atomicOr(&C.ctrl->err, (uint32_t)CE_TILE); return false; }
  rec = C.raw + a;
  rn = (uint32_t)(b - a);
  if (rn && rec[rn - 1u] == '\n') --rn;
  return true;
}

// ---- one record per thread, read in place
__device__ bool measure_in_place(const CleanParams& C, uint64_t r, uint64_t& bytes) {
  const uint8_t* rec = nullptr;
  uint32_t rn = 0;
  bytes = 0;
  bool keep = clean_frame(C, r, rec, rn);
  if (keep) keep = clean_record(C, rec, rn, [&](Bytes v) { bytes += v.n + 1ull; });  // a tab or the newline after every field
  if (keep && bytes >= (1ull << 32)) { atomicOr(&C.ctrl->err, (uint32_t)CE_TILE); keep = false; }
  return keep;
}

__device__ void write_in_place(const CleanParams& C, uint64_t r, uint64_t at) {
  const uint8_t* rec = nullptr;
  uint32_t rn = 0;
  if (!clean_frame(C, r, rec, rn)) return;
  uint8_t* dst = C.out + at;
  uint32_t k = 0;
  clean_record(C, rec, rn, [&](Bytes v) {
    for (uint32_t i = 0; i < v.n; ++i) dst[i] = v.p[i];
    dst += v.n;
    *dst++ = ++k < C.n_fields ? '\t' : '\n';
  });
}

// What the writing launch does once: the end of the offsets array, the size the caller needs, the
// capacity check.  Returns false (in every thread of every workgroup) when nothing may be written.
__device__ bool write_may_go_ahead(const CleanParams& C, bool first_thread) {
  if (C.ctrl->err) return false;
  if (first_thread) {
    C.out_off[C.total[1]] = C.total[0];
    C.ctrl->required = C.total[0];
    if (C.total[0] > C.out_cap) atomicOr(&C.ctrl->err, (uint32_t)CE_NOMEM);
  }
  return C.total[0] <= C.out_cap;
}

__device__ void measure_one(const CleanParams& C, uint64_t r) {
  uint64_t bytes = 0;
  const bool kept = measure_in_place(C, r, bytes);
  C.lens[r] = kept ? (uint32_t)bytes : 0u;
  C.lens[C.n_records + r] = kept ? 1u : 0u;
}
__device__ void write_one(const CleanParams& C, uint64_t r) {
  if (!C.lens[C.n_records + r]) return;
  C.out_off[C.base[C.n_records + r]] = C.base[r];
  write_in_place(C, r, C.base[r]);
}

__global__ __launch_bounds__(kBlock) void k_clean_measure(CleanParams C) {
  const uint64_t r = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (r < C.n_records) measure_one(C, r);
}

__global__ __launch_bounds__(kBlock) void k_clean_write(CleanParams C) {
  const uint64_t r = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (!write_may_go_ahead(C, r == 0)) return;
  if (r < C.n_records) write_one(C, r);
}

// ---- tiles of records staged in LDS
extern __shared__ __align__(16) uint8_t clean_smem[];

// Eight bytes at LDS position p (any alignment).
__device__ __forceinline__ void lds_window(uint32_t p, uint32_t& x0, uint32_t& x1) {
  const uint32_t* w = reinterpret_cast<const uint32_t*>(clean_smem);
  const uint32_t a = p >> 2, sh = (p & 3u) * 8u;
  const uint32_t w0 = w[a], w1 = w[a + 1], w2 = w[a + 2];
  x0 = __builtin_amdgcn_alignbit(w1, w0, sh);
  x1 = __builtin_amdgcn_alignbit(w2, w1, sh);
}
__device__ __forceinline__ bool lds_same(uint32_t p, uint32_t q, uint32_t n) {  // n bytes at p and at q
  for (uint32_t i = 0; i < n; i += 8u) {
    uint32_t a0, a1, b0, b1;
    lds_window(p + i, a0, a1);
    lds_window(q + i, b0, b1);
    const uint32_t m = n - i;
    const uint32_t m0 = m >= 4u ? ~0u : (1u << (8u * m)) - 1u, m1 = m <= 4u ? 0u : (m >= 8u ? ~0u : (1u << (8u * (m - 4u))) - 1u);
    if (((a0 ^ b0) & m0) | ((a1 ^ b1) & m1)) return false;
  }
  return true;
}
__device__ __forceinline__ uint32_t lds_find(uint32_t p, uint32_t e, uint32_t pat) {  // first byte of that kind in [p, e), or e
  while (p < e) {
    uint32_t x0, x1;
    lds_window(p, x0, x1);
    const uint32_t f0 = eq_flags(x0, pat), f1 = eq_flags(x1, pat);
    const uint32_t at = f0 ? ((uint32_t)__ffs((int)f0) - 1u) >> 3 : (f1 ? 4u + (((uint32_t)__ffs((int)f1) - 1u) >> 3) : 8u);
    p += at;
    if (at < 8u) break;
  }
  return p < e ? p : e;
}

// A cleaned field while its operators are applied: `n` bytes at LDS position `at`.
struct Field {
  uint32_t at, n;
};
// Two 16-bit numbers in a word (x low): LDS positions, and sizes inside a tile, all below 64 KiB.
__device__ __forceinline__ uint32_t two(uint32_t x, uint32_t y) { return x | (y << 16); }
__device__ __forceinline__ uint32_t lo16(uint32_t w) { return w & 0xffffu; }
__device__ __forceinline__ uint32_t hi16(uint32_t w) { return w >> 16; }

// The tile's text in whole 16-byte chunks, c-th chunk at raw + kCleanRawPad + 16 c; what lies outside the caller's buffer reads as zero.
__device__ __forceinline__ u32x4 text_chunk(uintptr_t ca, uintptr_t ok_lo, uintptr_t ok_hi) {
  u32x4 v;
  if (ca >= ok_lo && ca + 16u <= ok_hi) {
    v = *reinterpret_cast<const u32x4*>(ca);
  } else {
    uint32_t w[4] = {0, 0, 0, 0};
    for (uint32_t i = 0; i < 16; ++i) {
      const uintptr_t bi = ca + i;
      if (bi >= ok_lo && bi < ok_hi) w[i >> 2] |= (uint32_t)*reinterpret_cast<const uint8_t*>(bi) << (8u * (i & 3u));
    }
    v.x = w[0]; v.y = w[1]; v.z = w[2]; v.w = w[3];
  }
  return v;
}
// The same where all chunks lie inside the buffer (plain global loads: flat ones would also wait on the LDS counter).
using ChunkPtr = const __attribute__((address_space(1))) u32x4*;
__device__ __forceinline__ ChunkPtr chunks_at(uintptr_t a) { return reinterpret_cast<ChunkPtr>(a); }
// A table of the specification into LDS, all lanes taking part (sizes are whole words).
__device__ __forceinline__ void clean_table(uint32_t to, const void* from, uint32_t bytes) {
  for (uint32_t i = threadIdx.x; i < bytes / 4u; i += kCleanThreads)
    reinterpret_cast<uint32_t*>(clean_smem + to)[i] = reinterpret_cast<const uint32_t*>(from)[i];
}

// Measures tiles.  500,000 records of 826 bytes, 100 fields, 30 of them with operators, half of the records kept: both
// launches together 2.66 ms before (tables of all fields, twice; single-byte stores).
__global__ __launch_bounds__(kCleanThreads, kCleanWaves) void k_clean_measure_tile(CleanParams C) {
  __shared__ uint64_t s_off[kCleanMaxT + 1];
  __shared__ uint32_t s_len[kCleanMaxT], s_drop[kCleanMaxT];
  __shared__ uint32_t s_nseg[kCleanMaxT + 1];  // segments of a record, then the number of its first one
  __shared__ uint64_t s_out[kCleanMaxT];       // where the record starts in the tile's output
  __shared__ uint64_t s_total;
  __shared__ uint32_t s_bad;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t T = 1u << C.log2T, F = C.n_fields;
  uint8_t* raw = clean_smem;
  uint16_t* rows = reinterpret_cast<uint16_t*>(clean_smem + C.o_rows);
  uint32_t* fnew = reinterpret_cast<uint32_t*>(clean_smem + C.o_new);  // [n_of][T + 1] the cleaned field: position, bytes
  const OpField* of = reinterpret_cast<const OpField*>(clean_smem + C.o_of);
  const CleanOp* ops = reinterpret_cast<const CleanOp*>(clean_smem + C.o_ops);
  clean_table(C.o_args, C.args, C.args_bytes);  // (the newline at its end: see fbx_clean_create)
  clean_table(C.o_of, C.of, (C.n_of + 1u) * (uint32_t)sizeof(OpField));
  clean_table(C.o_ops, C.ops, C.n_ops * (uint32_t)sizeof(CleanOp));
  clean_table(C.o_keyed, C.keyed, C.n_keyed * 4u);
  const uint32_t* keyed = reinterpret_cast<const uint32_t*>(clean_smem + C.o_keyed);
  const uint32_t newline = C.o_args + C.args_bytes - 1u;
  // lanes that share a record: 256 / T, at most 64
  const uint32_t lg = 8u - C.log2T < 6u ? 8u - C.log2T : 6u;
  const uint32_t gsz = 1u << lg, j = tid & (gsz - 1u), rr = tid >> lg;
  const uintptr_t ok_lo = reinterpret_cast<uintptr_t>(C.raw), ok_hi = ok_lo + C.raw_len;
  // The next tile's record offsets are requested a tile ahead.  (Touching its text as well gains nothing: vector
  // instructions bound this kernel.)
  uint64_t off_next = 0;
  auto request_offsets = [&](uint32_t tile) {
    const uint64_t g = ((uint64_t)tile << C.log2T) + tid;
    if (tid <= T && g <= C.n_records) off_next = C.rec_off[g];
  };
  request_offsets(blockIdx.x * C.run);
  uint64_t run_bytes = 0, run_kept = 0;  // (of lane 63 of the first wavefront)
  const uint32_t first_tile = blockIdx.x * C.run, end_tile = min(first_tile + C.run, C.n_tiles);
  for (uint32_t tile = first_tile; tile < end_tile; ++tile) {
    const uint64_t g0 = (uint64_t)tile << C.log2T;
    const uint32_t nb = (uint32_t)min((uint64_t)T, C.n_records - g0);
    __syncthreads();  // (the sections are reused by the next tile)
    if (tid == 0) s_bad = 0;
    if (tid < kCleanMaxT) s_drop[tid] = 0;
    if (tid <= nb) s_off[tid] = off_next;
    __syncthreads();
    if (tid <= nb) {
      if (tid < nb) {
        const uint64_t a = off_next, b = s_off[tid + 1u];
        if (a > b || b > C.raw_len) atomicOr(&s_bad, (uint32_t)CE_OFFSETS);
        else if (b - a >= (1ull << 31)) atomicOr(&s_bad, (uint32_t)CE_TILE);
      }
    }
    __syncthreads();
    if (s_bad) {  // the call fails: the writing launch does nothing
      if (tid == 0) atomicOr(&C.ctrl->err, s_bad);
      break;
    }
    const uint64_t o0 = s_off[0];
    const uint32_t delta = (uint32_t)((ok_lo + o0) & 15u);
    const bool staged = s_off[nb] - o0 + delta <= (uint64_t)C.raw_cap;
    const bool act = staged && rr < nb;
    uint32_t rs = 0, re = 0, tabs = 0, content = 0, pads = 0, end_nl = 0;
    // What the operators changed in this lane's record.
    auto change = [&](uint32_t i, uint32_t& s, uint32_t& e, Field& f) -> bool {
      const uint16_t* rw = rows + rr * C.row_stride + of[i].field;
      s = (uint32_t)rw[0] + 1u;
      e = rw[1];
      if (e < s) e = s;
      const uint32_t w = fnew[i * (T + 1u) + rr];
      f = Field{lo16(w), hi16(w)};
      return f.n != e - s || (f.n && f.at != s);
    };
    if (staged) {
      {
        const uint32_t nchunks = (delta + (uint32_t)(s_off[nb] - o0) + 15u) >> 4;
        const uintptr_t a0 = ok_lo + o0 - delta;
        if (a0 >= ok_lo && a0 + 16ull * nchunks <= ok_hi) {  // whole chunks (all but the ends of the caller's buffer), four of a lane in flight
          constexpr uint32_t kInFlight = 4;
          const ChunkPtr from = chunks_at(a0);
          for (uint32_t c = tid; c < nchunks; c += kInFlight * kCleanThreads) {
            u32x4 v[kInFlight];
#pragma unroll
            for (uint32_t k = 0; k < kInFlight; ++k) v[k] = from[min(c + k * kCleanThreads, nchunks - 1u)];
#pragma unroll
            for (uint32_t k = 0; k < kInFlight; ++k)
              if (c + k * kCleanThreads < nchunks) *reinterpret_cast<u32x4*>(raw + kCleanRawPad + 16u * (c + k * kCleanThreads)) = v[k];
          }
        } else {
          for (uint32_t c = tid; c < nchunks; c += kCleanThreads)
            *reinterpret_cast<u32x4*>(raw + kCleanRawPad + 16u * c) = text_chunk(a0 + 16u * c, ok_lo, ok_hi);
        }
      }
      request_offsets(tile + 1u);
      __syncthreads();
      // field ends; entries from the record's tab count on hold its end
      if (act) {
        rs = kCleanRawPad + delta + (uint32_t)(s_off[rr] - o0);
        re = kCleanRawPad + delta + (uint32_t)(s_off[rr + 1] - o0);
        if (re > rs && raw[re - 1u] == '\n') { --re; end_nl = 1u; }  // one trailing newline is not part of the record
      }
      uint16_t* row = rows + rr * C.row_stride;
      tabs = split_bytes<false>(raw, rs, re, act, lg, j, kTabs, F, [&](uint32_t k, uint32_t pos) { row[1u + k] = (uint16_t)pos; }, 0u, 0u, [](uint32_t, uint32_t) {});
      if (act) {
        if (j == 0) row[0] = (uint16_t)(rs - 1u);
        for (uint32_t kk = tabs + j; kk < F; kk += gsz) row[1u + kk] = (uint16_t)re;
      }
      __syncthreads();
      // A key is looked up by all lanes of its record, eight bytes of the field a lane: pairs begin at the field's first
      // byte and after every ';', and the first one that begins with the name and a ':' is the one.  (A name with a
      // ':' or ';' in it is no key, see fbx_clean_create.  One lane a field, pair by pair, kept the other wavefronts
      // waiting: 145 of this launch's 357 us.)
      for (uint32_t q = 0; q < C.n_keyed; ++q) {
        const uint32_t i = keyed[q];
        const CleanOp op = ops[of[i].first_op];
        const uint32_t arg = C.o_args + op.arg_off, len = op.arg_len;
        uint32_t s = 0, e = 0, at = ~0u;
        if (act) {
          const uint16_t* rw = rows + rr * C.row_stride + of[i].field;
          s = (uint32_t)rw[0] + 1u;
          e = rw[1];
          auto is_it = [&](uint32_t p) -> bool { return p + len < e && raw[p + len] == ':' && lds_same(p, arg, len); };
          for (uint32_t p = s + 8u * j; p < e && at == ~0u; p += 8u * gsz) {
            if (p == s && is_it(p)) { at = p; break; }
            uint32_t x0, x1;
            lds_window(p, x0, x1);
            uint64_t f = ((uint64_t)eq_flags(x1, 0x3b3b3b3bu) << 32) | eq_flags(x0, 0x3b3b3b3bu);
            for (; f; f &= f - 1u) {
              const uint32_t c = p + ((uint32_t)__builtin_ctzll(f) >> 3) + 1u;
              if (is_it(c)) { at = c; break; }
            }
          }
        }
        for (uint32_t d = 1; d < gsz; d <<= 1) at = min(at, (uint32_t)__shfl_xor((int)at, (int)d, 64));
        if (act && j == 0) {
          const uint32_t v = at + len + 1u;
          fnew[i * (T + 1u) + rr] = at == ~0u ? two(s, 0u) : two(v, lds_find(v, e, 0x3b3b3b3bu) - v);
        }
      }
      if (C.n_keyed) __syncthreads();
      // lanes as (record, field with operators) pairs, the records of one field side by side: they run the same
      // operators (fields side by side had every wavefront walk the one keyed column with two lanes: 589 instead of
      // 409 vector instructions a record, both launches together)
      for (uint32_t pr = tid; pr < C.n_of << C.log2T; pr += kCleanThreads) {
        const uint32_t r = pr & (T - 1u), i = pr >> C.log2T;
        if (r >= nb) continue;
        const uint32_t k = of[i].field, o1 = of[i + 1u].first_op;
        const uint16_t* rw = rows + r * C.row_stride + k;
        const uint32_t s = (uint32_t)rw[0] + 1u, e = rw[1];
        Field f{s, e > s ? e - s : 0u};  // (a missing field is empty)
        uint32_t o = of[i].first_op;
        if (of[i].keyed) {
          const uint32_t w = fnew[i * (T + 1u) + r];
          f = Field{lo16(w), hi16(w)};
          ++o;
        }
        bool keep = true;
        for (; o < o1 && keep; ++o) {
          const CleanOp op = ops[o];
          const uint32_t arg = C.o_args + op.arg_off;
          if (op.kind == CK_FILL) {
            if (f.n == 0) f = Field{arg, op.arg_len};
          } else if (op.kind == CK_KEY) {
            // (not the field's first operator: pair by pair)
            const uint32_t fe = f.at + f.n;
            uint32_t p = f.at;
            for (;;) {
              if (p + op.arg_len < fe && raw[p + op.arg_len] == ':' && lds_same(p, arg, op.arg_len)) {
                const uint32_t v = p + op.arg_len + 1u;
                f = Field{v, lds_find(v, fe, 0x3b3b3b3bu) - v};
                break;
              }
              p = lds_find(p, fe, 0x3b3b3b3bu);
              if (p >= fe) { f.n = 0; break; }
              ++p;
            }
          } else if (op.kind == CK_KEEP) {
            keep = f.n >= op.arg_len && lds_same(f.at, arg, op.arg_len);
          } else {
            f.n = 0;  // a key that no pair can have
          }
        }
        if (!keep) s_drop[r] = 1u;
        fnew[i * (T + 1u) + r] = two(f.at, f.n);
      }
      __syncthreads();
      if (act) {
        content = (tabs >= F ? (uint32_t)rows[rr * C.row_stride + F] : re) - rs;  // (fields beyond the F-th are dropped)
        pads = tabs + 1u < F ? F - 1u - tabs : 0u;                                // (missing ones are empty)
        if (tabs >= F) end_nl = 0u;
      }
      uint32_t grow = 0, edits = 0;  // bytes the record grows by (modulo 2^32: it may shrink), fields that are replaced
      if (act && !s_drop[rr]) {
        for (uint32_t i = j; i < C.n_of; i += gsz) {
          uint32_t s, e;
          Field f;
          if (change(i, s, e, f)) { grow += f.n - (e - s); ++edits; }
        }
      }
      for (uint32_t d = 1; d < gsz; d <<= 1) {
        grow += __shfl_xor(grow, (int)d, 64);
        edits += __shfl_xor(edits, (int)d, 64);
      }
      if (act && j == 0) {
        s_len[rr] = content + pads + grow + 1u;
        s_nseg[rr] = s_drop[rr] ? 0u : 1u + 2u * edits + (pads ? 1u : 0u) + (end_nl && !pads ? 0u : 1u);
      }
    } else {
      if (tid < nb) {
        uint64_t n = 0;
        const bool kept = measure_in_place(C, g0 + tid, n);
        s_len[tid] = kept ? (uint32_t)n : 0u;
        s_drop[tid] = kept ? 0u : 1u;
        s_nseg[tid] = 0;
      }
      request_offsets(tile + 1u);
    }
    __syncthreads();
    if (wave == 0) {  // where records go inside the tile
      const bool kept = lane < nb && !s_drop[lane];
      const uint64_t mine = kept ? s_len[lane] : 0u;
      uint64_t len = mine;
      for (uint32_t d = 1; d < 64u; d <<= 1) {
        const uint64_t t = __shfl_up((unsigned long long)len, d, 64);
        if (lane >= d) len += t;
      }
      const uint32_t nseg = kept ? s_nseg[lane] : 0u;
      const uint32_t segs = group_prefix(nseg, 6u, lane);
      if (lane < nb) {
        s_out[lane] = len - mine;
        s_nseg[lane] = segs - nseg;
        C.rec_out[g0 + lane] = kept ? len - mine : kDropped;
      }
      const uint32_t n_kept = (uint32_t)__popcll(__ballot(kept));
      if (lane == 63u) {
        s_total = len;
        s_nseg[nb] = segs;
        // (a tile's output can be longer than its text: beyond 16-bit positions it is written in place)
        C.n_segs[tile] = staged && len <= 0xffffu ? segs : kInPlace;
        C.sums[tile] = len;
        run_bytes += len;
        run_kept += n_kept;
      }
    }
    __syncthreads();
    // segments of the records
    if (act && !s_drop[rr] && s_total <= 0xffffu) {
      uint32_t* seg = C.segs + g0 * (2ull * C.n_of + 3u);
      const uint32_t q0 = s_nseg[rr], out0 = (uint32_t)s_out[rr], len = s_len[rr];
      if (j == 0) {
        seg[q0] = two(out0, rs);
        if (!end_nl && !pads) seg[s_nseg[rr + 1u] - 1u] = two(out0 + len - 1u, newline);
      }
      if (!pads) {
        uint32_t grown = 0, done = 0;  // by the fields before this turn's
        for (uint32_t i0 = 0; i0 < C.n_of; i0 += gsz) {  // (the lanes of a group run the same number of turns)
          const uint32_t i = i0 + j;
          uint32_t s = 0, e = 0;
          Field f{0, 0};
          const bool ch = i < C.n_of && change(i, s, e, f);
          const uint32_t d = ch ? f.n - (e - s) : 0u;
          const uint32_t dp = group_prefix(d, lg, j), cp = group_prefix(ch ? 1u : 0u, lg, j);
          if (ch) {
            const uint32_t at = out0 + (s - rs) + grown + dp - d, q = q0 + 1u + 2u * (done + cp - 1u);
            seg[q] = two(at, f.at);
            seg[q + 1u] = two(at + f.n, e);
          }
          const int top = (int)(lane | (gsz - 1u));
          grown += __shfl(dp, top, 64);
          done += __shfl(cp, top, 64);
        }
      } else if (j == 0) {  // a record that lacks fields: its own come first, then tabs, between which fields may be filled
        uint32_t grown = 0, q = q0 + 1u;
        bool own = true;
        for (uint32_t i = 0; i < C.n_of; ++i) {
          uint32_t s, e;
          Field f;
          const uint32_t k = of[i].field;
          if (own && k > tabs) { seg[q++] = two(out0 + content + grown, kTabRun); own = false; }
          if (!change(i, s, e, f)) continue;
          const uint32_t at = out0 + grown + (own ? s - rs : content + (k - tabs));
          seg[q] = two(at, f.at);
          seg[q + 1u] = two(at + f.n, own ? e : kTabRun);
          q += 2u;
          grown += f.n - (e - s);
        }
        if (own) seg[q++] = two(out0 + content + grown, kTabRun);
        seg[q] = two(out0 + len - 1u, newline);
      }
    }
  }
  if (tid == 63u) {
    C.run_sums[blockIdx.x] = run_bytes;
    C.run_sums[gridDim.x + blockIdx.x] = run_kept;
  }
}

// Writes tiles.
__global__ __launch_bounds__(kCleanThreads, kCleanWaves) void k_clean_write_tile(CleanParams C) {
  __shared__ uint64_t s_wave[4][kCleanThreads / 64];
  __shared__ uint64_t s_off[kCleanMaxT + 1], s_out[kCleanMaxT];
  __shared__ uint32_t s_later, s_go;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t T = 1u << C.log2T;
  uint8_t* raw = clean_smem;
  uint32_t* seg = reinterpret_cast<uint32_t*>(clean_smem + C.o_seg);      // start in the tile's output, position in LDS
  uint16_t* later = reinterpret_cast<uint16_t*>(clean_smem + C.o_later);  // chunks of the output that cover several segments
  clean_table(C.o_args, C.args, C.args_bytes);
  if (tid == 0) s_go = C.ctrl->err ? 0u : 1u;
  uint64_t base = 0, n_before = 0, total = 0, n_total = 0;  // bytes and kept records: before this workgroup's tiles, of the batch
  for (uint32_t i = tid; i < gridDim.x; i += kCleanThreads) {
    const uint64_t n = C.run_sums[i], k = C.run_sums[gridDim.x + i];
    total += n;
    n_total += k;
    if (i < blockIdx.x) { base += n; n_before += k; }
  }
  auto over_workgroup = [&](uint64_t v, uint32_t row) -> uint64_t {
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor((unsigned long long)v, d, 64);
    if (lane == 0) s_wave[row][wave] = v;
    __syncthreads();
    v = 0;
    for (uint32_t w = 0; w < kCleanThreads / 64u; ++w) v += s_wave[row][w];
    return v;
  };
  base = over_workgroup(base, 0);
  n_before = over_workgroup(n_before, 1);
  total = over_workgroup(total, 2);
  n_total = over_workgroup(n_total, 3);
  const bool fits = total <= C.out_cap, go = fits && s_go != 0u;
  if (s_go && blockIdx.x == 0 && tid == 0) {
    __hip_atomic_store(const_cast<uint64_t*>(C.total), total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(const_cast<uint64_t*>(C.total) + 1, n_total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (fits) C.out_off[n_total] = total;
    else atomicOr(&C.ctrl->err, (uint32_t)CE_NOMEM);
  }
  const uintptr_t ok_lo = reinterpret_cast<uintptr_t>(C.raw), ok_hi = ok_lo + C.raw_len;
  const uint32_t* words = reinterpret_cast<const uint32_t*>(clean_smem);
  const uint32_t first_tile = blockIdx.x * C.run, end_tile = min(first_tile + C.run, C.n_tiles);
  for (uint32_t tile = first_tile; go && tile < end_tile; ++tile) {
    if (tid == 0) s_later = 0;
    const uint64_t g0 = (uint64_t)tile << C.log2T;
    const uint32_t nb = (uint32_t)min((uint64_t)T, C.n_records - g0);
    const uint32_t n_segs = C.n_segs[tile];
    const uint64_t total64 = C.sums[tile];
    if (tid <= nb) s_off[tid] = C.rec_off[g0 + tid];
    if (tid < nb) s_out[tid] = C.rec_out[g0 + tid];
    __syncthreads();
    const uint64_t kept = __ballot(lane < nb && s_out[lane] != kDropped);
    if (wave == 0 && ((kept >> lane) & 1ull)) C.out_off[n_before + (uint32_t)__popcll(kept & ((1ull << lane) - 1ull))] = base + s_out[lane];
    n_before += (uint32_t)__popcll(kept);
    if (n_segs == kInPlace) {
      if (tid < nb && s_out[tid] != kDropped) write_in_place(C, g0 + tid, base + s_out[tid]);
    } else if (total64) {
      // the text of the kept records, a wavefront a record, at the places the measuring launch had it
      const uint64_t o0 = s_off[0];
      const uint32_t delta = (uint32_t)((ok_lo + o0) & 15u);
      const uintptr_t a0 = ok_lo + o0 - delta;
      const uint32_t* segs = C.segs + g0 * (2ull * C.n_of + 3u);
      const uint32_t seg0 = tid < n_segs ? segs[tid] : 0u;  // (on its way together with the text)
      constexpr uint32_t kWaves = kCleanThreads / 64u, kInFlight = 4;
      static_assert(kWaves == 4u, "the mask of a wavefront's records below");
      // A bit per kept record that is this wavefront's, so that dropped ones cost nothing, however many there are (500,000 records
      // of 4 short fields, an eighth of them kept: 114 us a call where the places of every record were worked out, 98 so; of 16
      // fields 122 and 107, of 100 240 and 234; all kept, 4 fields, 129 and 114.  One record's text at a time: 105, 115, 246, 128).
      uint64_t mine = kept & (0x1111111111111111ull << __builtin_amdgcn_readfirstlane(wave));
      auto next = [&](uint32_t& c, uint32_t& c1) {  // this lane's first chunk of the next of them, and where the record's end
        c = c1 = 0;
        if (!mine) return;
        const uint32_t r = (uint32_t)__builtin_ctzll(mine);
        mine &= mine - 1u;
        c = ((delta + (uint32_t)(s_off[r] - o0)) >> 4) + lane;
        c1 = (delta + (uint32_t)(s_off[r + 1] - o0) + 15u) >> 4;
      };
      const bool inside = a0 >= ok_lo && a0 + (delta + (s_off[nb] - o0) + 16u) / 16u * 16u <= ok_hi;  // (one at least)
      if (inside) {  // whole chunks (all but the ends of the caller's buffer): the first ones of four records on their way at a time
        const ChunkPtr from = chunks_at(a0);
        while (mine) {
          u32x4 v[kInFlight];
          uint32_t c[kInFlight], c1[kInFlight];
#pragma unroll
          for (uint32_t k = 0; k < kInFlight; ++k) {
            next(c[k], c1[k]);
            v[k] = from[c[k] < c1[k] ? c[k] : 0u];
          }
#pragma unroll
          for (uint32_t k = 0; k < kInFlight; ++k) {
            if (c[k] < c1[k]) *reinterpret_cast<u32x4*>(raw + kCleanRawPad + 16u * c[k]) = v[k];
            for (uint32_t m = c[k] + 64u; m < c1[k]; m += 64u) *reinterpret_cast<u32x4*>(raw + kCleanRawPad + 16u * m) = from[m];
          }
        }
      } else {
        while (mine) {
          uint32_t c, c1;
          for (next(c, c1); c < c1; c += 64u) *reinterpret_cast<u32x4*>(raw + kCleanRawPad + 16u * c) = text_chunk(a0 + 16u * c, ok_lo, ok_hi);
        }
      }
      const uint32_t total = (uint32_t)total64;
      if (tid < n_segs) seg[tid] = seg0;
      for (uint32_t i = tid + kCleanThreads; i < n_segs; i += kCleanThreads) seg[i] = segs[i];
      if (tid == 0) seg[n_segs] = two(total, 0u);
      __syncthreads();
      // Lanes as 16-byte chunks of the output: chunk c holds the tile's bytes [16 c - shift, 16 c - shift + 16).  Most
      // lie inside one segment and are one shifted read and one store; the others (about one a segment) are put
      // aside and merged by lanes of their own, or every wavefront would merge for the sake of one or two lanes.
      const uintptr_t to = reinterpret_cast<uintptr_t>(C.out) + base;
      const uint32_t shift = (uint32_t)(to & 15u);
      uint8_t* dst0 = reinterpret_cast<uint8_t*>(to - shift);
      auto bytes16 = [&](uint32_t g, int32_t c0) -> u32x4 {  // what segment g puts at [c0, c0 + 16), were it that long
        u32x4 v;
        if (hi16(g) == kTabRun) {
          v.x = v.y = v.z = v.w = kTabs;
          return v;
        }
        const uint32_t p = hi16(g) + (uint32_t)(c0 - (int32_t)lo16(g));  // (16 bytes of padding lie before the text)
        const uint32_t at = p >> 2, sh = (p & 3u) * 8u;
        const uint32_t v0 = words[at], v1 = words[at + 1], v2 = words[at + 2], v3 = words[at + 3], v4 = words[at + 4];
        v.x = __builtin_amdgcn_alignbit(v1, v0, sh);
        v.y = __builtin_amdgcn_alignbit(v2, v1, sh);
        v.z = __builtin_amdgcn_alignbit(v3, v2, sh);
        v.w = __builtin_amdgcn_alignbit(v4, v3, sh);
        return v;
      };
      auto first_segment = [&](uint32_t lo) -> uint32_t {  // the last one that starts at lo or before
        uint32_t a = 0, b = n_segs - 1u;
        while (a < b) {
          const uint32_t mid = (a + b + 1u) >> 1;
          if (lo16(seg[mid]) <= lo) a = mid; else b = mid - 1u;
        }
        return a;
      };
      for (uint32_t c = tid; 16u * c < total + shift; c += kCleanThreads) {
        const int32_t c0 = (int32_t)(16u * c) - (int32_t)shift;
        const uint32_t a = first_segment(c0 < 0 ? 0u : (uint32_t)c0);
        if (c0 >= 0 && (uint32_t)c0 + 16u <= lo16(seg[a + 1u])) __builtin_nontemporal_store(bytes16(seg[a], c0), reinterpret_cast<u32x4*>(dst0 + 16u * (uint64_t)c));
        else later[atomicAdd(&s_later, 1u)] = (uint16_t)c;
      }
      __syncthreads();
      for (uint32_t i = tid; i < s_later; i += kCleanThreads) {
        const uint32_t c = later[i];
        const int32_t c0 = (int32_t)(16u * c) - (int32_t)shift;
        const uint32_t lo = c0 < 0 ? 0u : (uint32_t)c0, hi = min((uint32_t)(c0 + 16), total);
        uint32_t a = first_segment(lo);
        u32x4 w = bytes16(seg[a], c0);
        for (uint32_t next = lo16(seg[a + 1u]); next < hi; next = lo16(seg[a + 1u])) {
          const u32x4 x = bytes16(seg[++a], c0);
          const uint32_t skip = (uint32_t)((int32_t)next - c0);  // bytes of the chunk that earlier segments hold
          auto merge = [&](uint32_t old, uint32_t now, uint32_t first) {
            const uint32_t n = skip <= first ? 0u : min(skip - first, 4u);
            const uint32_t m = n >= 4u ? 0u : ~0u << (8u * n);
            return (old & ~m) | (now & m);
          };
          w.x = merge(w.x, x.x, 0u);
          w.y = merge(w.y, x.y, 4u);
          w.z = merge(w.z, x.z, 8u);
          w.w = merge(w.w, x.w, 12u);
        }
        uint8_t* dst = dst0 + 16u * (uint64_t)c;
        if (c0 >= 0 && c0 + 16 <= (int32_t)total) {
          __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(dst));
        } else {  // an end of the tile's output: its other bytes are the neighbours'
          for (uint32_t k = (uint32_t)((int32_t)lo - c0); k < (uint32_t)((int32_t)hi - c0); ++k) {
            const uint32_t v = k < 8u ? (k < 4u ? w.x : w.y) : (k < 12u ? w.z : w.w);
            dst[k] = (uint8_t)(v >> (8u * (k & 3u)));
          }
        }
      }
    }
    base += total64;
    __syncthreads();  // the sections are reused by the next tile
  }
  if (!C.export_to) return;
  // the last workgroup to finish hands control block and totals to the host (written by earlier launches or device-scope atomics)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) s_later = atomicAdd(&C.ctrl->finished, 1u) + 1u == gridDim.x ? 1u : 0u;
  __syncthreads();
  if (!s_later) return;
  constexpr uint32_t kCtrlWords = sizeof(Ctrl) / 8u;
  if (tid < kCtrlWords + 2u) {
    const uint64_t* from = tid < kCtrlWords ? reinterpret_cast<const uint64_t*>(C.ctrl) + tid : C.total + (tid - kCtrlWords);
    __hip_atomic_store(C.export_to + tid, __hip_atomic_load(from, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// The same without segments: for a scratch buffer of 24 bytes a record, and for specifications whose operators and
// arguments do not fit LDS beside the text.  A workgroup a tile, in both launches: lanes are (record, field) pairs that
// apply the field's operators (read from memory) and leave the cleaned field's length and source in LDS, a prefix sum per
// record turns lengths into positions, and the writing launch copies every field by single bytes, neighbouring lanes
// neighbouring fields.  300,000 records of 826 bytes: 1.63 ms, a thread a record 3.81 (a million by segments: 1.0).
struct Part {  // a cleaned field: `n` bytes at LDS position `at`, or at place `at` of the arguments (fixed)
  uint32_t at, n;
  bool fixed;
};
constexpr uint32_t kSrcConst = 0x80000000u;  // the field's bytes come from the arguments, not from the record
template <bool WRITE>
__global__ __launch_bounds__(kCleanThreads) void k_clean_tile(CleanParams C) {
  __shared__ uint64_t s_off[kCleanMaxT + 1];
  __shared__ uint64_t s_base[kCleanMaxT];
  __shared__ uint32_t s_rs[kCleanMaxT], s_re[kCleanMaxT], s_len[kCleanMaxT], s_drop[kCleanMaxT];
  __shared__ uint32_t s_bad;
  __shared__ uint32_t s_go;
  const uint32_t tid = threadIdx.x;
  if (WRITE) {  // (one thread decides for the workgroup: the error word may change while the launch runs)
    if (tid == 0) s_go = write_may_go_ahead(C, blockIdx.x == 0) ? 1u : 0u;
    __syncthreads();
    if (!s_go) return;
  }
  const uint32_t T = 1u << C.log2T, F = C.n_fields;
  const uint64_t g0 = (uint64_t)blockIdx.x << C.log2T;
  const uint32_t nb = (uint32_t)min((uint64_t)T, C.n_records - g0);
  uint8_t* raw = clean_smem;
  uint16_t* rows = reinterpret_cast<uint16_t*>(clean_smem + C.o_rows);
  uint32_t* flen = reinterpret_cast<uint32_t*>(clean_smem + C.o_len);  // bytes of the cleaned field and its separator, then where it starts in the cleaned record
  uint32_t* fsrc = reinterpret_cast<uint32_t*>(clean_smem + C.o_src);  // where its bytes come from
  if (tid == 0) s_bad = 0;
  if (tid <= nb) s_off[tid] = C.rec_off[g0 + tid];
  if (tid < kCleanMaxT) s_drop[tid] = 0;
  __syncthreads();
  if (tid < nb) {
    const uint64_t a = s_off[tid], b = s_off[tid + 1];
    if (a > b || b > C.raw_len) atomicOr(&s_bad, (uint32_t)CE_OFFSETS);
    else if (b - a >= (1ull << 31)) atomicOr(&s_bad, (uint32_t)CE_TILE);
  }
  __syncthreads();
  if (s_bad) {  // the call fails; the arrays the scan reads still get defined values
    if (tid == 0) atomicOr(&C.ctrl->err, s_bad);
    if (!WRITE && tid < nb) C.lens[g0 + tid] = C.lens[C.n_records + g0 + tid] = 0u;
    return;
  }
  const uint64_t o0 = s_off[0];
  const uintptr_t ok_lo = reinterpret_cast<uintptr_t>(C.raw), ok_hi = ok_lo + C.raw_len;
  const uint32_t delta = (uint32_t)((ok_lo + o0) & 15u);
  if (s_off[nb] - o0 + delta > (uint64_t)C.raw_cap) {  // the text does not fit the section
    if (tid < nb) {
      if (WRITE) write_one(C, g0 + tid); else measure_one(C, g0 + tid);
    }
    return;
  }
  {  // the tile's text, in whole 16-byte chunks
    const uint32_t nchunks = (delta + (uint32_t)(s_off[nb] - o0) + 15u) >> 4;
    const uintptr_t a0 = ok_lo + o0 - delta;
    for (uint32_t c = tid; c < nchunks; c += kCleanThreads)
      *reinterpret_cast<u32x4*>(raw + kCleanRawPad + 16u * c) = text_chunk(a0 + 16u * c, ok_lo, ok_hi);
    if (tid < nb) {
      s_rs[tid] = kCleanRawPad + delta + (uint32_t)(s_off[tid] - o0);
      s_re[tid] = kCleanRawPad + delta + (uint32_t)(s_off[tid + 1] - o0);
    }
  }
  __syncthreads();
  // field ends: 256 / T lanes (at most 64) share a record; entries from the record's tab count on hold its end
  const uint32_t lg = 8u - C.log2T < 6u ? 8u - C.log2T : 6u;
  const uint32_t gsz = 1u << lg, j = tid & (gsz - 1u), rr = tid >> lg;
  const bool act = rr < nb;
  uint32_t rs = 0, re = 0;
  if (act) {
    rs = s_rs[rr]; re = s_re[rr];
    if (re > rs && raw[re - 1u] == '\n') --re;  // one trailing newline is not part of the record
  }
  uint16_t* row = rows + rr * C.row_stride;
  {
    const uint32_t tabs = split_bytes<false>(raw, rs, re, act, lg, j, kTabs, F, [&](uint32_t k, uint32_t pos) { row[1u + k] = (uint16_t)pos; }, 0u, 0u, [](uint32_t, uint32_t) {});
    if (act) {
      if (j == 0) row[0] = (uint16_t)(rs - 1u);
      for (uint32_t kk = tabs + j; kk < F; kk += gsz) row[1u + kk] = (uint16_t)re;
    }
  }
  __syncthreads();
  // lanes as (record, field) pairs: a wavefront takes a record, its lanes the fields
  auto byte_of = [&](const Part& f, uint32_t i) -> uint32_t { return f.fixed ? C.args[f.at + i] : raw[f.at + i]; };
  for (uint32_t r = tid >> 6; r < nb; r += kCleanThreads / 64u) {
    const uint16_t* rw = rows + r * C.row_stride;
    for (uint32_t k = tid & 63u; k < F; k += 64u) {
      const uint32_t s = (uint32_t)rw[k] + 1u, e = rw[k + 1u];
      Part f{s, e > s ? e - s : 0u, false};  // (a missing field is empty)
      bool keep = true;
      for (uint32_t o = C.first_op[k]; o < C.first_op[k + 1] && keep; ++o) {
        const CleanOp op = C.ops[o];
        if (op.kind == CK_FILL) {
          if (f.n == 0) f = Part{op.arg_off, op.arg_len, true};
        } else if (op.kind == CK_KEY) {
          // value of the first pair "key:value" (pairs separated by ';') whose key is exactly the name
          uint32_t p = 0;
          for (;;) {
            uint32_t q = p;
            while (q < f.n && byte_of(f, q) != ';') ++q;
            uint32_t c = p;
            while (c < q && byte_of(f, c) != ':') ++c;
            if (c < q && c - p == op.arg_len) {
              bool same = true;
              for (uint32_t i = 0; i < op.arg_len && same; ++i) same = byte_of(f, p + i) == C.args[op.arg_off + i];
              if (same) { f.at += c + 1u; f.n = q - c - 1u; break; }
            }
            if (q >= f.n) { f.n = 0; break; }
            p = q + 1u;
          }
        } else if (op.kind == CK_NONE) {
          f.n = 0;
        } else {
          keep = f.n >= op.arg_len;
          for (uint32_t i = 0; i < op.arg_len && keep; ++i) keep = byte_of(f, i) == C.args[op.arg_off + i];
        }
      }
      if (!keep) s_drop[r] = 1u;
      flen[r * F + k] = f.n + 1u;  // a tab or the newline after every field
      fsrc[r * F + k] = f.at | (f.fixed ? kSrcConst : 0u);
    }
  }
  __syncthreads();
  {  // lengths become positions inside the cleaned record: the lanes that shared the record's tabs share its fields
    const uint32_t c = (F + gsz - 1u) >> lg;
    const uint32_t k0 = min(j * c, F), k1 = min(k0 + c, F);
    uint32_t sum = 0;
    if (act) for (uint32_t k = k0; k < k1; ++k) sum += flen[rr * F + k];
    const uint32_t incl = group_prefix(sum, lg, j);
    const uint32_t total = __shfl(incl, (int)(lane_id() | (gsz - 1u)), 64);
    if (act) {
      uint32_t at = incl - sum;
      for (uint32_t k = k0; k < k1; ++k) {
        const uint32_t n = flen[rr * F + k];
        flen[rr * F + k] = at;
        at += n;
      }
      if (j == 0) s_len[rr] = total;
    }
  }
  __syncthreads();
  if (!WRITE) {
    if (tid < nb) {
      const bool kept = !s_drop[tid];
      C.lens[g0 + tid] = kept ? s_len[tid] : 0u;
      C.lens[C.n_records + g0 + tid] = kept ? 1u : 0u;
    }
    return;
  }
  if (tid < nb && !s_drop[tid]) {
    const uint64_t at = C.base[g0 + tid];
    s_base[tid] = at;
    C.out_off[C.base[C.n_records + g0 + tid]] = at;
  }
  __syncthreads();
  for (uint32_t r = tid >> 6; r < nb; r += kCleanThreads / 64u) {
    if (s_drop[r]) continue;
    for (uint32_t k = tid & 63u; k < F; k += 64u) {
      const uint32_t at = flen[r * F + k];
      const uint32_t n = (k + 1u < F ? flen[r * F + k + 1u] : s_len[r]) - at - 1u;
      const uint32_t src = fsrc[r * F + k];
      uint8_t* dst = C.out + s_base[r] + at;
      if (src & kSrcConst) {
        const uint8_t* from = C.args + (src & ~kSrcConst);
        for (uint32_t i = 0; i < n; ++i) dst[i] = from[i];
      } else {
        const uint8_t* from = raw + src;
        for (uint32_t i = 0; i < n; ++i) dst[i] = from[i];
      }
      dst[n] = k + 1u < F ? '\t' : '\n';
    }
  }
}

// Before the tile kernels, one launch: control block, totals, and the specification's tables, which
// travel with the launch's arguments when they fit (otherwise the host has enqueued a copy of its own).
constexpr uint32_t kImageInline = 3584;
template <uint32_t N>
struct ImageArgs { uint32_t w[N / 4]; };
template <uint32_t N>
__global__ __launch_bounds__(kBlock) void k_clean_setup(Ctrl* ctrl, uint64_t* total, uint32_t* tables, uint32_t table_words, ImageArgs<N> image) {
  const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i == 0) { Ctrl c = {}; *ctrl = c; total[0] = total[1] = 0; }
  if (i < table_words) tables[i] = image.w[i];
}

constexpr size_t kMaxExports = 16;  // calls at the same time that get host memory to export to (further ones copy)

uint64_t up256(uint64_t x) { return (x + 255u) & ~uint64_t(255); }

int hex_digit(char c) {
  if (c >= '0' && c <= '9') return c - '0';
  if (c >= 'a' && c <= 'f') return c - 'a' + 10;
  if (c >= 'A' && c <= 'F') return c - 'A' + 10;
  return -1;
}

thread_local std::string g_clean_create_error;

}  // namespace

namespace {
// A tile's LDS: text, tables, and all of it (without asking for more than the 64 KiB that every workgroup gets; positions
// in the text and the arguments behind it are 16-bit).
constexpr uint64_t kTextMax = 24576, kTableMax = 32768, kLdsMax = 62000;
}  // namespace

struct fbx_clean {
  uint32_t n_fields = 0;
  std::vector<CleanOp> ops;          // sorted by field (stable)
  std::vector<uint32_t> first_op;    // n_fields + 1
  std::vector<uint8_t> args;
  std::vector<uint8_t> image;        // ops, first_op, args, and what only the tile kernels read, as they lie in the scratch
  uint64_t core = 0;                 // bytes up to the end of args
  uint64_t off_ops = 0, off_first = 0, off_args = 0, off_of = 0, off_keyed = 0;
  std::vector<uint32_t> keyed;       // entries of the table of fields with operators whose first one looks a key up
  uint32_t n_of = 0, args_bytes = 0;

  // LDS for tiles of T records: tables of the kernels that keep segments, what those need beside for any T (operators and
  // arguments), and the tables of the kernel that keeps none.
  uint64_t row_stride() const { return (n_fields + 2ull + 7ull) & ~uint64_t(7); }
  uint64_t segments(uint64_t T) const { return T * (2ull * n_of + 3) + 1; }
  uint64_t tables(uint64_t T) const { return std::max<uint64_t>(T * row_stride() * 2 + (T + 1) * n_of * 4ull, segments(T) * 6 + 16); }
  uint64_t fixed() const { return args_bytes + 16 + (n_of + 1) * sizeof(OpField) + ops.size() * sizeof(CleanOp) + keyed.size() * 4 + 128; }
  uint64_t plain_tables(uint64_t T) const { return T * (row_stride() * 2 + n_fields * 8ull); }
  // whether tiles of some size keep segments, whatever the records' length
  bool keeps_segments() const { return tables(1) <= kTableMax && kTextMax + tables(1) + fixed() <= kLdsMax; }

  // Several threads may run one specification at the same time: what calls leave here is under the lock.
  std::mutex lock;
  std::vector<uint64_t*> exports, idle;  // host memory that the tile kernel writes control block and totals to: all there is, and what no call uses
  int grid_dev = -1;
  uint32_t grid_lds = 0, grid = 0;   // workgroups of the measuring kernel that run at the same time on that device with that much LDS
  std::string error;
};

namespace {

void clean_error(fbx_clean& c, const std::string& why) {
  std::lock_guard<std::mutex> hold(c.lock);
  c.error = why;
}

// Host memory for the sizes of one call, its own until the call is over: two calls at the same time must not read each
// other's.  None (a copy is enqueued instead) when there is none to be had or kMaxExports calls have theirs.
uint64_t* export_taken(fbx_clean& c) {
  std::lock_guard<std::mutex> hold(c.lock);
  if (c.idle.empty() && c.exports.size() < kMaxExports) {
    void* mem = nullptr;
    if (hipHostMalloc(&mem, sizeof(Ctrl) + 16, hipHostMallocPortable) == hipSuccess) {
      c.exports.push_back(static_cast<uint64_t*>(mem));
      c.idle.push_back(static_cast<uint64_t*>(mem));
    } else {
      (void)hipGetLastError();
    }
  }
  if (c.idle.empty()) return nullptr;
  uint64_t* mine = c.idle.back();
  c.idle.pop_back();
  return mine;
}
void export_returned(fbx_clean& c, uint64_t* mem) {
  std::lock_guard<std::mutex> hold(c.lock);
  c.idle.push_back(mem);
}

// Workgroups of the measuring kernel that run at the same time (the LDS decides): asked once per device and size.
uint32_t clean_grid(fbx_clean& c, uint32_t lds) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); dev = 0; }
  std::lock_guard<std::mutex> hold(c.lock);
  if (c.grid_dev != dev || c.grid_lds != lds) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(&k_clean_measure_tile), kCleanThreads, lds) != hipSuccess || per_cu < 1) {
      (void)hipGetLastError();
      per_cu = 1;
    }
    c.grid_dev = dev;
    c.grid_lds = lds;
    c.grid = std::min(kMaxRuns, tile_cu_count() * static_cast<uint32_t>(per_cu));
  }
  return c.grid;
}

struct CleanLayout {
  uint64_t ctrl, total, tables;
  uint64_t lens, base, part;                                // one record per thread
  uint64_t run_sums, sums, n_segs, rec_out, segs, end;      // tiles (in the same place)
};

// small: no segments are kept (24 bytes a record; with them it is 20 and 4 for each that a record can have).
CleanLayout clean_layout(const fbx_clean& c, uint64_t n, bool small) {
  CleanLayout L{};
  uint64_t o = 0;
  L.ctrl = o; o = up256(o + sizeof(Ctrl));
  L.total = o; o = up256(o + 16);
  L.tables = o; o = up256(o + (small ? c.core : c.image.size()));
  const uint64_t shared = o;
  L.lens = o; o = up256(o + 2 * n * 4);
  L.base = o; o = up256(o + 2 * n * 8);
  L.part = o; o = up256(o + 2ull * scan_segments(static_cast<uint32_t>(n)) * 8);
  L.end = o;
  if (small) return L;
  o = shared;
  L.run_sums = o; o = up256(o + 2ull * kMaxRuns * 8);
  L.sums = o; o = up256(o + n * 8);                         // (a tile has a record at least)
  L.n_segs = o; o = up256(o + n * 4);
  L.rec_out = o; o = up256(o + n * 8);
  L.segs = o; o = up256(o + n * (2ull * c.n_of + 3) * 4);
  L.end = std::max(L.end, o);
  return L;
}

}  // namespace

extern "C" {

fbx_status fbx_clean_create(const char* spec, size_t spec_len, fbx_clean** out) {
  if (!spec || !out) { g_clean_create_error = "spec and out must not be NULL"; return FBX_E_ARG; }
  std::unique_ptr<fbx_clean> c(new (std::nothrow) fbx_clean());
  if (!c) return FBX_E_ARG;
  std::vector<CleanOp> in_spec_order;
  const std::string text(spec, spec_len);
  size_t pos = 0;
  int line_no = 0;
  bool header = false;
  auto fail = [&](const std::string& why) {
    g_clean_create_error = "line " + std::to_string(line_no) + ": " + why;
    return FBX_E_SPEC;
  };
  while (pos <= text.size()) {
    size_t nl = text.find('\n', pos);
    if (nl == std::string::npos) nl = text.size();
    std::string line = text.substr(pos, nl - pos);
    pos = nl + 1;
    ++line_no;
    const size_t hash = line.find('#');
    if (hash != std::string::npos) line.resize(hash);
    std::vector<std::string> words;
    for (size_t i = 0; i < line.size();) {
      while (i < line.size() && (line[i] == ' ' || line[i] == '\t' || line[i] == '\r')) ++i;
      size_t j = i;
      while (j < line.size() && line[j] != ' ' && line[j] != '\t' && line[j] != '\r') ++j;
      if (j > i) words.push_back(line.substr(i, j - i));
      i = j;
    }
    if (words.empty()) continue;
    if (!header) {
      if (words.size() != 2 || words[0] != "fbxclean" || words[1] != "1") return fail("expected 'fbxclean 1'");
      header = true;
      continue;
    }
    if (words[0] == "fields") {
      char* end = nullptr;
      const unsigned long f = words.size() == 2 ? strtoul(words[1].c_str(), &end, 10) : 0;
      if (words.size() != 2 || *end || f == 0 || f > 65535 || c->n_fields) return fail("bad or repeated 'fields'");
      c->n_fields = static_cast<uint32_t>(f);
      continue;
    }
    CleanOp op{};
    const char* arg_key = nullptr;
    if (words[0] == "fill") { op.kind = CK_FILL; arg_key = "value"; }
    else if (words[0] == "key") { op.kind = CK_KEY; arg_key = "name"; }
    else if (words[0] == "keep") { op.kind = CK_KEEP; arg_key = "prefix"; }
    if (!op.kind || !c->n_fields) return fail("unknown operator, or an operator before 'fields'");
    bool have_field = false, have_arg = false;
    for (size_t w = 1; w < words.size(); ++w) {
      const size_t eq = words[w].find('=');
      if (eq == std::string::npos) return fail("expected key=value");
      const std::string key = words[w].substr(0, eq), val = words[w].substr(eq + 1);
      if (key == "field" && !have_field) {
        char* end = nullptr;
        const unsigned long f = strtoul(val.c_str(), &end, 10);
        if (val.empty() || *end || f >= c->n_fields) return fail("field out of range");
        op.field = static_cast<uint32_t>(f);
        have_field = true;
      } else if (key == arg_key && !have_arg) {
        if (val.size() % 2 || val.size() / 2 > 255) return fail("bytes are written as an even number of hex digits, at most 255 bytes");
        op.arg_off = static_cast<uint32_t>(c->args.size());
        op.arg_len = static_cast<uint32_t>(val.size() / 2);
        for (size_t i = 0; i < val.size(); i += 2) {
          const int hi = hex_digit(val[i]), lo = hex_digit(val[i + 1]);
          if (hi < 0 || lo < 0) return fail("bad hex digit");
          const uint8_t b = static_cast<uint8_t>(hi * 16 + lo);
          if (op.kind == CK_FILL && (b == '\t' || b == '\n')) return fail("a fill value holds no tab and no newline");
          c->args.push_back(b);
        }
        have_arg = true;
      } else {
        return fail("unknown or repeated key '" + key + "'");
      }
    }
    if (!have_field || !have_arg) return fail("missing key");
    if (op.kind == CK_FILL && op.arg_len == 0) return fail("a fill value is not empty");
    if (op.kind == CK_KEY)  // (a pair's key ends at its first ':', a pair at the first ';')
      for (uint32_t i = 0; i < op.arg_len; ++i)
        if (c->args[op.arg_off + i] == ':' || c->args[op.arg_off + i] == ';') { op.kind = CK_NONE; break; }
    in_spec_order.push_back(op);
  }
  if (!header || !c->n_fields) { ++line_no; return fail("missing header or 'fields'"); }
  c->ops = in_spec_order;
  std::stable_sort(c->ops.begin(), c->ops.end(), [](const CleanOp& a, const CleanOp& b) { return a.field < b.field; });
  c->first_op.assign(c->n_fields + 1, 0);
  for (const CleanOp& op : c->ops) ++c->first_op[op.field + 1];
  for (uint32_t k = 0; k < c->n_fields; ++k) c->first_op[k + 1] += c->first_op[k];
  std::vector<OpField> of;
  for (uint32_t k = 0; k < c->n_fields; ++k)
    if (c->first_op[k + 1] > c->first_op[k]) {
      const bool key = c->ops[c->first_op[k]].kind == CK_KEY;
      if (key) c->keyed.push_back(static_cast<uint32_t>(of.size()));
      of.push_back(OpField{k, c->first_op[k], key ? 1u : 0u});
    }
  c->n_of = static_cast<uint32_t>(of.size());
  of.push_back(OpField{c->n_fields, static_cast<uint32_t>(c->ops.size()), 0u});
  uint64_t o = 0;
  c->off_ops = o; o += c->ops.size() * sizeof(CleanOp);
  c->off_first = o; o += c->first_op.size() * 4;
  c->off_args = o; c->core = o + c->args.size();
  c->args.resize(c->args.size() / 4 * 4 + 4, '\n');  // whole words, the last byte a newline
  c->args_bytes = static_cast<uint32_t>(c->args.size());
  o += c->args.size();
  c->off_of = o; o += of.size() * sizeof(OpField);
  c->off_keyed = o; o += c->keyed.size() * 4;
  c->image.assign(o, 0);
  if (!c->ops.empty()) std::memcpy(c->image.data() + c->off_ops, c->ops.data(), c->ops.size() * sizeof(CleanOp));
  std::memcpy(c->image.data() + c->off_of, of.data(), of.size() * sizeof(OpField));
  if (!c->keyed.empty()) std::memcpy(c->image.data() + c->off_keyed, c->keyed.data(), c->keyed.size() * 4);
  std::memcpy(c->image.data() + c->off_args, c->args.data(), c->args.size());
  std::memcpy(c->image.data() + c->off_first, c->first_op.data(), c->first_op.size() * 4);
  *out = c.release();
  return FBX_OK;
}

void fbx_clean_destroy(fbx_clean* clean) {
  if (!clean) return;
  for (uint64_t* mem : clean->exports) (void)hipHostFree(mem);
  delete clean;
}

const char* fbx_clean_last_error(const fbx_clean* clean) { return clean ? clean->error.c_str() : g_clean_create_error.c_str(); }

fbx_status fbx_clean_scratch_hint(const fbx_clean* clean, uint64_t n_records, uint64_t* bytes) {
  if (!clean || !bytes || n_records >= (1ull << 32)) return FBX_E_ARG;
  *bytes = clean_layout(*clean, n_records, !clean->keeps_segments()).end;  // (no room for segments that no kernel would keep)
  return FBX_OK;
}

fbx_status fbx_clean_run(fbx_clean* clean, const uint8_t* d_raw, uint64_t raw_len, const uint64_t* d_rec_off,
                         uint64_t n_records, uint8_t* d_out, uint64_t out_cap, uint64_t* d_out_off, void* d_scratch,
                         uint64_t scratch_bytes, void* hip_stream, fbx_clean_result* out) {
  if (!clean || !out || !d_rec_off || (!d_raw && raw_len) || !d_out_off || (!d_out && out_cap) || !d_scratch) {
    if (clean) clean_error(*clean, "NULL argument");
    return FBX_E_ARG;
  }
  if (n_records >= (1ull << 32) || (reinterpret_cast<uintptr_t>(d_scratch) & 255u)) {
    clean_error(*clean, "a call takes fewer than 2^32 records and a 256-byte aligned scratch buffer");
    return FBX_E_ARG;
  }
  const bool can_keep = clean->keeps_segments();
  CleanLayout L = clean_layout(*clean, n_records, !can_keep);
  out->n_kept = out->out_len = 0;
  out->required_scratch = L.end;
  const bool small = !can_keep || scratch_bytes < L.end;  // (a buffer without room for the tiles' segments still does, for kernels that keep none)
  const bool short_of = can_keep && small;
  if (small && scratch_bytes < clean_layout(*clean, n_records, true).end) {
    clean_error(*clean, "scratch buffer too small: need " + std::to_string(L.end) + " bytes");
    return FBX_E_NOMEM;
  }
  if (small) L = clean_layout(*clean, n_records, true);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint8_t* sc = static_cast<uint8_t*>(d_scratch);
  auto hip_failed = [&](hipError_t e, const char* where) {
    clean_error(*clean, std::string(where) + ": " + hipGetErrorString(e));
    (void)hipGetLastError();
    return FBX_E_HIP;
  };
  Ctrl* ctrl = reinterpret_cast<Ctrl*>(sc + L.ctrl);
  uint64_t* total = reinterpret_cast<uint64_t*>(sc + L.total);
  CleanParams C{};
  C.raw = d_raw; C.raw_len = raw_len; C.rec_off = d_rec_off; C.n_records = n_records;
  C.ops = reinterpret_cast<const CleanOp*>(sc + L.tables + clean->off_ops);
  C.first_op = reinterpret_cast<const uint32_t*>(sc + L.tables + clean->off_first);
  C.of = reinterpret_cast<const OpField*>(sc + L.tables + clean->off_of);
  C.keyed = reinterpret_cast<const uint32_t*>(sc + L.tables + clean->off_keyed);
  C.n_keyed = static_cast<uint32_t>(clean->keyed.size());
  C.args = sc + L.tables + clean->off_args;
  C.n_fields = clean->n_fields; C.n_of = clean->n_of; C.n_ops = static_cast<uint32_t>(clean->ops.size());
  C.args_bytes = clean->args_bytes;
  C.lens = reinterpret_cast<uint32_t*>(sc + L.lens);
  C.base = reinterpret_cast<const uint64_t*>(sc + L.base);
  C.total = total;
  C.out = d_out; C.out_cap = out_cap; C.out_off = d_out_off; C.ctrl = ctrl;
  // Tiles: as many records as usually fit the text section with room to spare, their tables within the budget.  Segments
  // are kept where there is room for them in the scratch buffer and for operators and arguments in LDS: five times as
  // fast as going without (500,000 records of 826 bytes: 0.52 against 2.7 ms).
  const uint64_t mean = n_records ? raw_len / n_records + 1 : 1;
  auto text = [&](uint64_t T) { return std::min<uint64_t>(kTextMax, std::max<uint64_t>(4096, (T * mean * (small ? 6 : 5) / 4 + 64 + 15) & ~uint64_t(15))); };
  auto fits = [&](uint64_t T) {
    if (small) return clean->plain_tables(T) <= kTableMax;
    return clean->tables(T) <= kTableMax && text(T) + clean->tables(T) + clean->fixed() <= kLdsMax;
  };
  uint32_t log2T = 6;
  while (log2T && ((mean << log2T) * 5 / 4 > kTextMax || !fits(1ull << log2T))) --log2T;
  const bool tiles = n_records && fits(1ull << log2T);
  uint32_t lds_measure = 0, lds_write = 0;
  if (tiles) {
    const uint64_t T = 1ull << log2T;
    auto up16 = [](uint64_t x) { return static_cast<uint32_t>((x + 15u) & ~uint64_t(15)); };
    C.log2T = log2T;
    C.raw_cap = static_cast<uint32_t>(text(T));
    C.row_stride = static_cast<uint32_t>(clean->row_stride());
    const uint32_t text_end = kCleanRawPad + C.raw_cap + 16;  // (the splitter reads whole 16-byte chunks: one more behind the text)
    if (small) {
      C.o_rows = text_end;
      C.o_len = static_cast<uint32_t>(C.o_rows + T * C.row_stride * 2);
      C.o_src = static_cast<uint32_t>(C.o_len + T * clean->n_fields * 4);
      lds_measure = lds_write = static_cast<uint32_t>(C.o_src + T * clean->n_fields * 4);
    } else {
      C.o_args = text_end;
      const uint32_t behind = up16(C.o_args + clean->args_bytes + 16);
      C.o_rows = behind;
      C.o_new = up16(C.o_rows + T * C.row_stride * 2);
      C.o_of = up16(C.o_new + (T + 1) * clean->n_of * 4);
      C.o_ops = up16(C.o_of + (clean->n_of + 1) * sizeof(OpField));
      C.o_keyed = up16(C.o_ops + C.n_ops * sizeof(CleanOp));
      lds_measure = up16(C.o_keyed + clean->keyed.size() * 4) + 16;
      C.o_seg = behind;
      // (a chunk that covers several segments holds the end of one of them: no more chunks than those and the two ends)
      C.o_later = up16(C.o_seg + clean->segments(T) * 4);
      lds_write = up16(C.o_later + (clean->segments(T) + 1) * 2) + 16;
      C.run_sums = reinterpret_cast<uint64_t*>(sc + L.run_sums);
      C.sums = reinterpret_cast<uint64_t*>(sc + L.sums);
      C.n_segs = reinterpret_cast<uint32_t*>(sc + L.n_segs);
      C.rec_out = reinterpret_cast<uint64_t*>(sc + L.rec_out);
      C.segs = reinterpret_cast<uint32_t*>(sc + L.segs);
    }
    C.n_tiles = static_cast<uint32_t>((n_records + T - 1) >> log2T);
  }
  struct { Ctrl c; uint8_t pad[256 - sizeof(Ctrl)]; uint64_t total[2]; } back;
  static_assert(sizeof(back) == 256 + 16, "read-back layout");
  // set-up: the tables go along as arguments of the launch if they are small
  const uint64_t image_bytes = small ? (clean->core + 3) & ~uint64_t(3) : clean->image.size();  // (whole words)
  const bool inl = image_bytes <= kImageInline;
  hipError_t e = hipSuccess;
  if (!inl) e = hipMemcpyAsync(sc + L.tables, clean->image.data(), image_bytes, hipMemcpyHostToDevice, st);
  if (e == hipSuccess) {
    ImageArgs<kImageInline> image;
    if (inl) std::memcpy(image.w, clean->image.data(), image_bytes);
    const uint32_t table_words = inl ? static_cast<uint32_t>(image_bytes / 4) : 0u;
    hipLaunchKernelGGL(k_clean_setup<kImageInline>, dim3((table_words + kBlock) / kBlock), dim3(kBlock), 0, st, ctrl, total,
                       reinterpret_cast<uint32_t*>(sc + L.tables), table_words, image);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return hip_failed(e, "set-up");
  if (tiles && !small) {
    // as many workgroups as run at the same time, each a run of tiles; the writing launch takes the same runs
    const uint32_t at_once = clean_grid(*clean, lds_measure);
    C.run = (C.n_tiles + at_once - 1) / at_once;
    const uint32_t grid = (C.n_tiles + C.run - 1) / C.run;
    hipLaunchKernelGGL(k_clean_measure_tile, dim3(grid), dim3(kCleanThreads), lds_measure, st, C);
    e = hipGetLastError();
    if (e == hipSuccess) C.export_to = export_taken(*clean);
    if (e == hipSuccess) hipLaunchKernelGGL(k_clean_write_tile, dim3(grid), dim3(kCleanThreads), lds_write, st, C);
    if (e == hipSuccess) e = hipGetLastError();
  } else {
    const uint32_t blocks = tiles ? C.n_tiles : static_cast<uint32_t>((n_records + kBlock - 1) / kBlock);
    if (n_records) {
      if (tiles) hipLaunchKernelGGL(k_clean_tile<false>, dim3(blocks), dim3(kCleanThreads), lds_measure, st, C);
      else hipLaunchKernelGGL(k_clean_measure, dim3(blocks), dim3(kBlock), 0, st, C);
      e = hipGetLastError();
      if (e == hipSuccess)
        e = launch_scan(C.lens, reinterpret_cast<uint64_t*>(sc + L.base), total, reinterpret_cast<uint64_t*>(sc + L.part), 2,
                        static_cast<uint32_t>(n_records), ctrl, st);
      if (e != hipSuccess) return hip_failed(e, "measuring and placing records");
    }
    if (tiles) hipLaunchKernelGGL(k_clean_tile<true>, dim3(blocks), dim3(kCleanThreads), lds_write, st, C);
    else hipLaunchKernelGGL(k_clean_write, dim3(std::max(blocks, 1u)), dim3(kBlock), 0, st, C);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return hip_failed(e, "cleaning records");
  if (!C.export_to) e = hipMemcpyAsync(&back, sc + L.ctrl, sizeof back, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_failed(e, "read-back");
  if (C.export_to) {
    std::memcpy(&back.c, C.export_to, sizeof back.c);
    std::memcpy(back.total, C.export_to + sizeof(Ctrl) / 8, sizeof back.total);
    export_returned(*clean, C.export_to);  // (after an error of the runtime it stays out of use: a kernel may still write it)
  }
  if (back.c.err & CE_OFFSETS) { clean_error(*clean, "record offsets must be non-decreasing and end within raw_len"); return FBX_E_INPUT; }
  if (back.c.err & CE_TILE) { clean_error(*clean, "a record of 2 GiB or more, or one that cleans to 4 GiB or more"); return FBX_E_INPUT; }
  out->n_kept = back.total[1];
  out->out_len = back.total[0];
  if (back.c.err & CE_NOMEM) {
    clean_error(*clean, "output buffer too small: need " + std::to_string(back.total[0]) + " bytes");
    return FBX_E_NOMEM;
  }
  clean_error(*clean, !short_of ? "" : "the scratch buffer holds no segments: " + std::to_string(out->required_scratch) + " bytes make the call faster");
  return FBX_OK;
}

}  // extern "C"
