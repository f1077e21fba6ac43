// Splitting staged bytes at a delimiter with groups of lanes (Section 5 of the paper, first
// paragraph: a record is split at its delimiter before anything else happens to it), shared by the
// tile kernel of the extraction path and by the cleaning stage.  Device code for gfx950 only.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace fbx {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The thread's number, hidden from the optimiser's view of the loops around the caller: what
// follows from it (lane masks, per-lane addresses) is then worked out where it is used instead
// of once per kernel, where each such value would hold a register for good.
__device__ __forceinline__ uint32_t thread_id() {
  uint32_t t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
__device__ __forceinline__ uint32_t lane_id() { return thread_id() & 63u; }

// 0x80 in exactly the bytes of w that equal the byte repeated in pat.
__device__ __forceinline__ uint32_t eq_flags(uint32_t w, uint32_t pat) {
  const uint32_t x = w ^ pat;
  return ~(((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x | 0x7f7f7f7fu);
}
constexpr uint32_t kTabs = 0x09090909u, kCommas = 0x2c2c2c2cu;

// Inclusive prefix sum of v inside groups of 1 << lg neighbouring lanes (j: the lane's number in
// its group).  Inside a row of 16 lanes the steps of 1, 2, 4 and 8 lanes are single
// data-parallel-primitive moves (row_shr, zero for a lane without a source); a group of several
// rows then adds the totals of its earlier rows, which come through the LDS crossbar.  Every
// lane of the wavefront must call it.
template <int D>
__device__ __forceinline__ uint32_t row_shr(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x110 + D, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t group_prefix(uint32_t v, uint32_t lg, uint32_t j) {
  if (lg >= 1u) { const uint32_t t = row_shr<1>(v); v += j >= 1u ? t : 0u; }
  if (lg >= 2u) { const uint32_t t = row_shr<2>(v); v += j >= 2u ? t : 0u; }
  if (lg >= 3u) { const uint32_t t = row_shr<4>(v); v += j >= 4u ? t : 0u; }
  if (lg >= 4u) { const uint32_t t = row_shr<8>(v); v += j >= 8u ? t : 0u; }
  if (lg > 4u) {  // groups of two or four rows: add the totals of the group's rows before the lane's own
    const uint32_t first = lane_id() - j;
    uint32_t carry = 0;
    for (uint32_t k = 1; k < (1u << (lg - 4u)); ++k) {
      const uint32_t t = __shfl(v, (int)(first + 16u * k - 1u), 64);
      if ((j >> 4) >= k) carry += t;
    }
    v += carry;
  }
  return v;
}

// Bit i of the result: byte i of the sixteen is NOT the byte repeated in pat (a byte below 0x80).
// With the top bits out of the way, (w ^ pat) + 0x7f carries into the top bit of every byte that
// differs; a dot product with the weights 1, 2, 4 ... packs the top bits (0x7f or 0xff a byte; the
// 0x7f parts sum up to a constant that the accumulator starts from): four vector instructions a
// word and class, one of them shared between the classes that are looked for in the same text.
__device__ __forceinline__ uint32_t differs16(const u32x4& w, const u32x4& low7, uint32_t pat) {
  auto top = [&](uint32_t x, uint32_t l) -> uint32_t { return ((l ^ pat) + 0x7f7f7f7fu) | x | 0x7f7f7f7fu; };
  uint32_t lo = __builtin_amdgcn_udot4(top(w.x, low7.x), 0x08040201u, 0u - 127u * 255u, false);
  lo = __builtin_amdgcn_udot4(top(w.y, low7.y), 0x80402010u, lo, false);
  uint32_t hi = __builtin_amdgcn_udot4(top(w.z, low7.z), 0x08040201u, 0u - 127u * 255u, false);
  hi = __builtin_amdgcn_udot4(top(w.w, low7.w), 0x80402010u, hi, false);
  return ((hi << 8) + lo) >> 7;
}

// 1 << lg neighbouring lanes of a wavefront (j = 0 .. (1 << lg) - 1) split the staged
// bytes [rs, re) at every delimiter (pat_a: the delimiter in all four bytes) and, with TWO,
// find those of a second kind in the same walk.  Each lane takes an equal run of the 16-byte
// chunks that cover the range and counts its delimiters; a prefix sum over the group turns the
// counts into ordinals, and a second walk calls emit_a(k, position) for the k-th delimiter,
// k < limit_a (and emit_b, limit_b).  Returns the number of delimiters in the whole range, those
// of the second kind times 2^16 added (a range holds fewer than 2^16 bytes).  Every lane of a
// group calls it; those with act == false emit nothing.
template <bool TWO, class EmitA, class EmitB>
__device__ __forceinline__ uint32_t split_bytes(const uint8_t* raw, uint32_t rs, uint32_t re, bool act, uint32_t lg, uint32_t j,
                                                uint32_t pat_a, uint32_t limit_a, EmitA&& emit_a, uint32_t pat_b, uint32_t limit_b,
                                                EmitB&& emit_b) {
  const uint32_t gsz = 1u << lg;
  const uint32_t ab = rs & ~15u;
  const uint32_t nc = (act && re > rs) ? (re - ab + 15u) >> 4 : 0u;  // 16-byte chunks that cover the range
  const uint32_t c = (nc + gsz - 1u) >> lg;                          // chunks per lane
  const uint32_t c0 = min(j * c, nc), c1 = min(c0 + c, nc);
  // One bit per byte, for 64 bytes at a time: bit i is set when byte i of the piece (which starts at chunk q0) is a
  // delimiter of the range and of this lane's run.
  struct Piece { uint32_t a0, a1, b0, b1; };
  auto piece = [&](uint32_t q0) -> Piece {
    uint32_t na0 = ~0u, na1 = ~0u, nb0 = ~0u, nb1 = ~0u;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      if (q0 + q < c1) {
        const u32x4 w = *reinterpret_cast<const u32x4*>(raw + ab + 16u * (q0 + q));
        u32x4 low7;
        low7.x = w.x & 0x7f7f7f7fu; low7.y = w.y & 0x7f7f7f7fu; low7.z = w.z & 0x7f7f7f7fu; low7.w = w.w & 0x7f7f7f7fu;
        const uint32_t da = differs16(w, low7, pat_a);
        if (q == 0) na0 = da | 0xffff0000u;
        else if (q == 1) na0 = (na0 & 0xffffu) | (da << 16);
        else if (q == 2) na1 = da | 0xffff0000u;
        else na1 = (na1 & 0xffffu) | (da << 16);
        if (TWO) {
          const uint32_t db = differs16(w, low7, pat_b);
          if (q == 0) nb0 = db | 0xffff0000u;
          else if (q == 1) nb0 = (nb0 & 0xffffu) | (db << 16);
          else if (q == 2) nb1 = db | 0xffff0000u;
          else nb1 = (nb1 & 0xffffu) | (db << 16);
        }
      }
    }
    Piece m{0u, 0u, 0u, 0u};
    if (q0 < c1) {  // (the piece starts before re)
      const uint32_t p = ab + 16u * q0;
      const uint32_t lo = rs > p ? rs - p : 0u, hi = min(re - p, 64u);
      const uint64_t in = (hi >= 64u ? ~0ull : (1ull << hi) - 1ull) & (~0ull << lo);
      m.a0 = ~na0 & (uint32_t)in;
      m.a1 = ~na1 & (uint32_t)(in >> 32);
      if (TWO) {
        m.b0 = ~nb0 & (uint32_t)in;
        m.b1 = ~nb1 & (uint32_t)(in >> 32);
      }
    }
    return m;
  };
  auto count = [](const Piece& m) -> uint32_t { return __popc(m.a0) + __popc(m.a1) + (TWO ? (__popc(m.b0) + __popc(m.b1)) << 16 : 0u); };
  // A lane's first two pieces (128 bytes, all there is in all but very long records) are kept for the second walk.
  const Piece first = piece(c0);
  uint32_t cnt = count(first);
  Piece second{0u, 0u, 0u, 0u};
  if (c > 4u) {
    second = piece(c0 + 4u);
    cnt += count(second);
    for (uint32_t q = c0 + 8u; q < c1; q += 4u) cnt += count(piece(q));
  }
  const uint32_t incl = group_prefix(cnt, lg, j);
  const uint32_t total = __shfl(incl, (int)(lane_id() | (gsz - 1u)), 64);
  if (!act) return total;
  uint32_t ka = (incl - cnt) & 0xffffu, kb = (incl - cnt) >> 16;
  auto walk = [&](uint32_t m, uint32_t base, uint32_t& k, uint32_t limit, auto&& emit) {
    for (uint32_t n = min((uint32_t)__popc(m), k < limit ? limit - k : 0u); n; --n) {
      emit(k, base + (uint32_t)__builtin_ctz(m));  // (m is not zero here)
      ++k;
      m &= m - 1u;
    }
  };
  auto walk_piece = [&](const Piece& m, uint32_t q0) {
    const uint32_t base = ab + 16u * q0;
    walk(m.a0, base, ka, limit_a, emit_a);
    walk(m.a1, base + 32u, ka, limit_a, emit_a);
    if (TWO) {
      walk(m.b0, base, kb, limit_b, emit_b);
      walk(m.b1, base + 32u, kb, limit_b, emit_b);
    }
  };
  walk_piece(first, c0);
  if (c > 4u) {
    walk_piece(second, c0 + 4u);
    for (uint32_t q = c0 + 8u; q < c1; q += 4u) walk_piece(piece(q), q);
  }
  return total;
}

}  // namespace
}  // namespace fbx
