// Tiled per-leaf and value-level copies: records whose leaves differ in size
// (Sec. 1 record dimension), SPLIT views (Sec. 3) against a partner of another
// form, and pairs that convert value by value (two computed views, integer
// ChangeType, bit-packed codes over 32 bits).  Both sides in one
// linearisation order; AoSoA blocks that fit a tile.
//
// One workgroup takes one tile of records.  The source's tile is a set of
// contiguous segments (the records of an AoS or AoSoA part, a run of each
// plane, byte column or bit stream): they come into LDS with direct 16-byte
// loads, 1 KiB per wave instruction, all in flight at once.  Then the leaves
// are taken one after another: consecutive lanes read consecutive records of
// the leaf from LDS, convert, and store to the destination.  Every property of
// a leaf is wave-uniform and comes through scalar loads, so the branches on it
// are scalar.  Where both sides keep 16 bytes of a leaf together, a lane
// moves 16 bytes.  Bit-packed codes are ORed into stream words in LDS, and
// records without padding are put together there; both leave in 16-byte
// stores after the last leaf.
//
// Half of a wave's cycles wait for memory: a tile's loads, leaves and stores
// follow each other.  Scalar issue takes 21-44 % of the time and vector issue
// 11-48 %, so what a wave decodes per leaf is kept short (the plan holds each
// leaf's addresses and steps ready, a wave takes a leaf over hundreds of records,
// K = 8 records a lane share the branches; with the branches taken per record the
// same copies were up to 2.4 times slower).  A store instruction that covers part
// of a line costs the whole line's write unless the other parts reach L2 at once:
// hence the images, and the waves working on the leaves of the same records
// together (padded AoS records: 130 MB written for 120 MB of lines, 413 MB with
// the leaves one after another).  Such records' stores leave holes in every line:
// waves wait 57 % of their cycles to issue, against 15-30 % elsewhere, and the
// copy moves 3.6 TB/s (stored by full dwords and bytes from an image, with half
// the requests, it took the same time).
//
// 5 Mi records {u8, f64, i16, f32} (150 MB moved a copy) in 27-37 us, padded
// AoS destinations in 57-64 us; one thread per record and leaf took 77-114 us.
// 3 Mi records of 3 integers between i32, i16 and 12-bit codes in 20-25 us, one
// thread per 32 records took 130-237 us.  (K = 4: 8 Mi records of 7 leaves into
// AoS 87 us, K = 8 70; the other copies within 5 %.)
#include "value_codec.hpp"

namespace lm {

namespace {

struct Spec {
  uint32_t kind, lsz, bits, E, M, form, flag;
};

__device__ __forceinline__ Spec spec_of(uint32_t w) {
  return {w & 3u, (w >> 2) & 3u, (w >> 4) & 127u, (w >> 11) & 15u, (w >> 15) & 63u, (w >> 21) & 7u, (w >> 24) & 1u};
}

// A leaf's place on one side: the offset of tile-local record r, r * step
// (planar, AoS), or by blocks of L records (AoSoA; BLK).
struct Place {
  uint32_t step, L, block;
  Div div_L;
};

template <bool BLK>
__device__ __forceinline__ uint32_t place(const Place& p, uint32_t r) {
  if (!BLK || p.L == 0u) return r * p.step;
  const uint32_t q = fdiv(r, p.div_L);
  return q * p.block + (r - q * p.L) * p.step;
}

// The values of one leaf for K records a lane, 64 apart.
constexpr uint32_t K = 8;
constexpr uint32_t kStep = 64u * K;  // records per wave and pass

// Element of B bytes at LDS address a, at any alignment.
template <uint32_t B>
__device__ __forceinline__ uint64_t lds_elem(const uint8_t* lds, uint32_t a) {
  if constexpr (B == 1u) return lds[a];
  // aligned dwords around it (slots end with 16 bytes of slack) and byte shifts
  const uint32_t* p = (const uint32_t*)(lds + (a & ~3u));
  const uint32_t sh = a & 3u;
  const uint32_t d0 = p[0], d1 = p[1];
  const uint32_t lo = __builtin_amdgcn_alignbyte(d1, d0, sh);
  if constexpr (B == 2u) return lo & 0xFFFFu;
  if constexpr (B == 4u) return lo;
  return (uint64_t)lo | ((uint64_t)__builtin_amdgcn_alignbyte(p[2], d1, sh) << 32);
}

// 16 bytes at LDS address a, at any alignment.
__device__ __forceinline__ u32x4 lds_16(const uint8_t* lds, uint32_t a) {
  if ((a & 15u) == 0u) return *(const u32x4*)(lds + a);
  const uint32_t* p = (const uint32_t*)(lds + (a & ~3u));
  const uint32_t d0 = p[0], d1 = p[1], d2 = p[2], d3 = p[3];
  if ((a & 3u) == 0u) return u32x4{d0, d1, d2, d3};
  const uint32_t d4 = p[4], sh = a & 3u;
  return u32x4{__builtin_amdgcn_alignbyte(d1, d0, sh), __builtin_amdgcn_alignbyte(d2, d1, sh),
               __builtin_amdgcn_alignbyte(d3, d2, sh), __builtin_amdgcn_alignbyte(d4, d3, sh)};
}

// Reads elements whose LDS addresses are multiples of their size (`plain`),
// or of any alignment.
template <typename T>
__device__ __forceinline__ void read_elems(const uint8_t* lds, const uint32_t (&at)[K], bool plain, uint64_t (&v)[K]) {
  if (plain) {
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) v[k] = *(const T*)(lds + at[k]);
  } else {
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) v[k] = lds_elem<sizeof(T)>(lds, at[k]);
  }
}

// Stored bits of a leaf for the lane's K records.
template <int OPS, bool BLK>
__device__ __forceinline__ void tree_read(const TreeArgs& a, const Spec& s, const Place& pl, uint32_t col,
                                          uint32_t base, const uint8_t* lds, const uint32_t (&r)[K], uint64_t (&v)[K]) {
  if (s.kind == TR_ELEM) {
    uint32_t at[K];
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) at[k] = base + place<BLK>(pl, r[k]);
    const bool plain = ((base | pl.step | (BLK ? pl.block : 0u)) & ((1u << s.lsz) - 1u)) == 0u;
    switch (s.lsz) {
      case 0: read_elems<uint8_t>(lds, at, true, v); break;
      case 1: read_elems<uint16_t>(lds, at, plain, v); break;
      case 2: read_elems<uint32_t>(lds, at, plain, v); break;
      default: read_elems<uint64_t>(lds, at, plain, v); break;
    }
    return;
  }
  if constexpr (OPS > 0) {
    if (s.kind == TR_BITS) {
      const uint32_t* w = (const uint32_t*)(lds + base);
      if (s.bits <= 32u) {
        const uint32_t mask = s.bits >= 32u ? 0xFFFFFFFFu : (1u << s.bits) - 1u;
#pragma unroll
        for (uint32_t k = 0; k < K; ++k) {
          const uint32_t bit = r[k] * s.bits, q = bit >> 5;
          v[k] = __builtin_amdgcn_alignbit(w[q + 1u], w[q], bit & 31u) & mask;
        }
      } else {
        const uint64_t mask = s.bits >= 64u ? ~0ull : (1ull << s.bits) - 1ull;
#pragma unroll
        for (uint32_t k = 0; k < K; ++k) {
          const uint32_t bit = r[k] * s.bits, q = bit >> 5, sh = bit & 31u;
          const uint32_t d1 = w[q + 1u];
          v[k] = ((uint64_t)__builtin_amdgcn_alignbit(d1, w[q], sh) |
                  ((uint64_t)__builtin_amdgcn_alignbit(w[q + 2u], d1, sh) << 32)) & mask;
        }
      }
      return;
    }
  }
#pragma unroll
  for (uint32_t k = 0; k < K; ++k) v[k] = 0ull;
  if (s.kind == TR_BYTES)
    for (uint32_t j = 0; j < (1u << s.lsz); ++j) {
      const uint32_t c = col + j, cb = (a.scol[c >> 1] >> (16u * (c & 1u))) & 0xFFFFu;
#pragma unroll
      for (uint32_t k = 0; k < K; ++k) v[k] |= (uint64_t)lds[cb + place<BLK>(pl, r[k])] << (8u * j);
    }
}

// One element to an address of any alignment (the hardware takes it).
template <typename T>
__device__ __forceinline__ void put(uint8_t* p, T v) {
  __builtin_memcpy(p, &v, sizeof(T));
}

// FULL: all K records of every lane are in the tile.
template <typename T, bool BLK, bool FULL>
__device__ __forceinline__ void write_elems(uint8_t* base, const Place& pl, const uint32_t (&r)[K], uint32_t nt,
                                            const uint64_t (&v)[K]) {
#pragma unroll
  for (uint32_t k = 0; k < K; ++k)
    if (FULL || r[k] < nt) put<T>(base + place<BLK>(pl, r[k]), (T)v[k]);
}

// The same into the LDS image of a record-major destination.
template <typename T, bool FULL>
__device__ __forceinline__ void write_image(uint8_t* lds, uint32_t base, uint32_t step, const uint32_t (&r)[K],
                                            uint32_t nt, const uint64_t (&v)[K]) {
  const bool plain = ((base | step) & (sizeof(T) - 1u)) == 0u;
#pragma unroll
  for (uint32_t k = 0; k < K; ++k) {
    if (!FULL && r[k] >= nt) continue;
    uint8_t* p = lds + base + r[k] * step;
    if (plain) {
      *(T*)p = (T)v[k];
    } else {
#pragma unroll
      for (uint32_t j = 0; j < sizeof(T); ++j) p[j] = (uint8_t)(v[k] >> (8u * j));
    }
  }
}

template <int OPS, bool BLK, bool FULL>
__device__ __forceinline__ void tree_write(const TreeArgs& a, const Spec& d, const Place& pl, uint32_t col,
                                           uint8_t* base, uint8_t* lds, uint32_t img, const uint32_t (&r)[K],
                                           uint32_t nt, const uint64_t (&v)[K]) {
  if (d.kind == TR_ELEM) {
    if (img) {
      switch (d.lsz) {
        case 0: write_image<uint8_t, FULL>(lds, img, pl.step, r, nt, v); break;
        case 1: write_image<uint16_t, FULL>(lds, img, pl.step, r, nt, v); break;
        case 2: write_image<uint32_t, FULL>(lds, img, pl.step, r, nt, v); break;
        default: write_image<uint64_t, FULL>(lds, img, pl.step, r, nt, v); break;
      }
      return;
    }
    switch (d.lsz) {
      case 0: write_elems<uint8_t, BLK, FULL>(base, pl, r, nt, v); break;
      case 1: write_elems<uint16_t, BLK, FULL>(base, pl, r, nt, v); break;
      case 2: write_elems<uint32_t, BLK, FULL>(base, pl, r, nt, v); break;
      default: write_elems<uint64_t, BLK, FULL>(base, pl, r, nt, v); break;
    }
    return;
  }
  if constexpr (OPS > 0) {
    if (d.kind == TR_BITS) {
      uint32_t* words = (uint32_t*)(lds + img);
      const uint64_t mask = d.bits < 64u ? (1ull << d.bits) - 1ull : ~0ull;
#pragma unroll
      for (uint32_t k = 0; k < K; ++k) {
        if (!FULL && r[k] >= nt) continue;
        const uint64_t c = v[k] & mask;
        const uint32_t bit = r[k] * d.bits, sh = bit & 31u;
        uint32_t* w = words + (bit >> 5);
        const uint32_t lo = (uint32_t)c;
        __hip_atomic_fetch_or(w, lo << sh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (sh + d.bits > 32u)
          __hip_atomic_fetch_or(w + 1, (uint32_t)(c >> (32u - sh)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (sh + d.bits > 64u)
          __hip_atomic_fetch_or(w + 2, (uint32_t)(c >> 32) >> (32u - sh), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      return;
    }
  }
  // byte columns: `base` lies as far into column `col` as the others' runs into theirs
  const uint64_t off = (uint64_t)(base - a.dcol[col]);
  for (uint32_t j = 0; j < (1u << d.lsz); ++j) {
    uint8_t* cb = a.dcol[col + j] + off;
#pragma unroll
    for (uint32_t k = 0; k < K; ++k)
      if (FULL || r[k] < nt) cb[place<BLK>(pl, r[k])] = (uint8_t)(v[k] >> (8u * j));
  }
}

__device__ __forceinline__ uint32_t ext32(uint32_t v, uint32_t bits, bool sgn) {
  const uint32_t sh = 32u - bits;
  return sgn ? (uint32_t)((int32_t)(v << sh) >> sh) : (v << sh) >> sh;
}

__device__ __forceinline__ uint64_t ext64(uint64_t v, uint32_t bits, bool sgn) {
  const uint32_t sh = 64u - bits;
  return sgn ? (uint64_t)((int64_t)(v << sh) >> sh) : (v << sh) >> sh;
}

// Stored bits of a float leaf -> the leaf's own format, and back: the
// conversions of ChangeType and the codes of BitPackedFloatSoA.
__device__ __forceinline__ uint32_t load_f32(uint64_t v, const Spec& s) {
  switch (s.form) {
    case TF_CODE: return dec_f32((uint32_t)v, s.E, s.M);
    case TF_F16: return (uint32_t)widen<5, 10, 8, 23>(v);
    case TF_BF16: return (uint32_t)widen<8, 7, 8, 23>(v);
    case TF_F64: return cvt_f64_f32(v);
    default: return (uint32_t)v;
  }
}

__device__ __forceinline__ uint64_t store_f32(uint32_t v, const Spec& d) {
  switch (d.form) {
    case TF_CODE: return d.flag ? enc_f32_rne(v, d.E, d.M) : enc_f32(v, d.E, d.M);
    case TF_F16: return cvt_f32_f16(v);
    case TF_BF16: return cvt_f32_bf16(v);
    case TF_F64: return cvt_f32_f64(v);
    default: return v;
  }
}

__device__ __forceinline__ uint64_t load_f64(uint64_t v, const Spec& s) {
  switch (s.form) {
    case TF_CODE: return dec_f64((uint32_t)v, s.E, s.M);
    case TF_F16: return widen<5, 10, 11, 52>(v);
    case TF_BF16: return widen<8, 7, 11, 52>(v);
    case TF_F32: return cvt_f32_f64((uint32_t)v);
    default: return v;
  }
}

__device__ __forceinline__ uint64_t store_f64(uint64_t v, const Spec& d) {
  switch (d.form) {
    case TF_CODE: return d.flag ? enc_f64_rne(v, d.E, d.M) : enc_f64(v, d.E, d.M);
    case TF_F16: return narrow_rne<11, 52, 5, 10>(v);
    case TF_BF16: return narrow_rne<11, 52, 8, 7>(v);
    case TF_F32: return cvt_f64_f32(v);
    default: return v;
  }
}

__device__ __forceinline__ uint32_t form_type(uint32_t form) {
  return form == TF_F16 ? LLAMA_F16 : form == TF_BF16 ? LLAMA_BF16 : form == TF_F32 ? LLAMA_F32 : LLAMA_F64;
}

// Any float leaf (type ut) through the run-time codecs.
__device__ __forceinline__ uint64_t gen_value(uint64_t v, const Spec& s, const Spec& d, uint32_t ut) {
  uint32_t E, M;
  gen_float_fmt(ut, E, M);
  if (s.form == TF_CODE) v = gen_widen(v, s.E, s.M, E, M, false);
  else if (s.form != TF_RAW) v = gen_convert(v, form_type(s.form), ut);
  if (d.form == TF_CODE) v = gen_narrow(v, E, M, d.E, d.M, d.flag != 0u);
  else if (d.form != TF_RAW) v = gen_convert(v, ut, form_type(d.form));
  return v;
}

template <int OPS>
__device__ __forceinline__ void tree_value(const Spec& s, const Spec& d, uint32_t what, uint64_t (&v)[K]) {
  const uint32_t op = (what >> 16) & 15u, ut = (what >> 20) & 15u, ub = (what >> 24) & 127u;
  const bool us = (what >> 31) != 0u;
  if (OPS == 0 || op == TO_MOVE) return;
  if (op == TO_INT32) {
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) v[k] = ext32(ext32((uint32_t)v[k], s.bits, s.flag != 0u), ub, us);
    return;
  }
  if (op == TO_F32) {
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) v[k] = store_f32(load_f32(v[k], s), d);
    return;
  }
  if constexpr (OPS > 1) {
    if (op == TO_INT64) {
#pragma unroll
      for (uint32_t k = 0; k < K; ++k) v[k] = ext64(ext64(v[k], s.bits, s.flag != 0u), ub, us);
    } else if (op == TO_F64) {
#pragma unroll
      for (uint32_t k = 0; k < K; ++k) v[k] = store_f64(load_f64(v[k], s), d);
    } else {
#pragma unroll
      for (uint32_t k = 0; k < K; ++k) v[k] = gen_value(v[k], s, d, ut);
    }
  }
}

// A leaf whose 16-byte runs stay together on both sides: 16 / size records
// per lane; the tile's last, partial run byte by byte.
template <bool BLK>
__device__ __forceinline__ void move_runs(const Place& sp, const Place& dp, uint32_t sbase, uint8_t* base,
                                          uint32_t lsz, const uint8_t* lds, uint32_t r0, uint32_t r1) {
  const uint32_t V = 16u >> lsz;
  for (uint32_t r = r0 + lane_id() * V; r < r1; r += 64u * V) {
    const uint32_t at = sbase + place<BLK>(sp, r);
    uint8_t* p = base + place<BLK>(dp, r);
    if (r + V <= r1) {
      put<u32x4>(p, lds_16(lds, at));
    } else {
      for (uint32_t k = 0; k < (r1 - r) << lsz; ++k) p[k] = lds[at + k];
    }
  }
}

// One leaf over the records [r0, r1) of the tile, by one wave.
template <int OPS, bool BLK>
__device__ __forceinline__ void tree_leaf(const TreeArgs& a, const TreeLeaf& lf, const Place& sp, const Place& dp,
                                          uint8_t* base, uint8_t* lds, uint32_t r0, uint32_t r1) {
  const Spec s = spec_of(lf.src), d = spec_of(lf.dst);
  const uint32_t sc = lf.what & 255u, dc = (lf.what >> 8) & 255u, op = (lf.what >> 16) & 15u;
  const uint32_t sbase = lf.lds & 0xFFFFu, img = lf.lds >> 16;
  if (op == TO_MOVE && s.kind == TR_ELEM && d.kind == TR_ELEM && !img) {
    const uint32_t V = 16u >> s.lsz;
    auto runs = [&](const Place& p) { return p.step == 1u << s.lsz && (!BLK || p.L == 0u || (p.L & (V - 1u)) == 0u); };
    if (runs(sp) && runs(dp)) {
      move_runs<BLK>(sp, dp, sbase, base, s.lsz, lds, r0, r1);
      return;
    }
  }
  for (uint32_t rr = r0; rr < r1; rr += kStep) {
    uint32_t r[K], rc[K];
    uint64_t v[K];
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) {
      r[k] = rr + 64u * k + lane_id();
      rc[k] = r[k] < r1 ? r[k] : r1 - 1u;
    }
    tree_read<OPS, BLK>(a, s, sp, sc, sbase, lds, rc, v);
    tree_value<OPS>(s, d, lf.what, v);
    if (rr + kStep <= r1) tree_write<OPS, BLK, true>(a, d, dp, dc, base, lds, img, r, r1, v);
    else tree_write<OPS, BLK, false>(a, d, dp, dc, base, lds, img, r, r1, v);
  }
}

}  // namespace

// OPS 0: moves only; 1: and integers of 32 bits and f32 leaves; 2: all.
template <int OPS>
__global__ __launch_bounds__(kThreads) void k_tree(const TreeArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const uint32_t t = blockIdx.x;
  const uint64_t i0 = (uint64_t)t * a.tile;
  const uint64_t left = a.n - i0;
  const uint32_t nt = left < (uint64_t)a.tile ? (uint32_t)left : a.tile;
  const uint32_t lane = lane_id(), nw = num_waves();
  // source segments -> LDS: the waves take the 1 KiB groups of all segments in turn
  uint32_t turn = wave_id();
  for (uint32_t q = 0; q < a.nseg; ++q) {
    const TreeSeg sg = a.seg[q];
    const uint32_t bits = sg.what & 8191u, L = (sg.what >> 13) & 8191u, phase = sg.lds & 15u;
    const uint32_t nr = L > 1u && nt < a.tile ? (nt + L - 1u) / L * L : nt;  // AoSoA: whole blocks
    const uint32_t bytes = phase + ((nr * bits + 7u) >> 3);  // from the aligned base
    const uint32_t len = (bytes + 3u) & ~3u;
    const uint64_t start = (i0 >> 3) * bits;  // tiles are multiples of 128 records
    // bytes that can be read: 128 records more are 16 bytes more; past the last
    // tile's only what the blob still has
    const uint32_t end = bytes + (left >= a.tile + 128ull ? 16u : left == nt ? sg.what >> 26 : 0u);
    const auto rs = make_rsrc(sg.base + start, end);
    const uint32_t groups = (len + 1023u) >> 10;
    uint32_t grp = turn;
    for (; grp < groups; grp += nw) {
      const uint32_t off = grp * 1024u + lane * 16u;
      if (off < len) {
        if (off + 16u <= end) {
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(lds + (sg.lds & ~15u) + grp * 1024u), 16, off, 0, 0, kLoadStream);
        } else {  // across the end
          load_tail16(rs, off, end - off, lds + (sg.lds & ~15u) + off);
        }
      }
    }
    turn = grp - groups;  // the wave's first group of the next segment
  }
  if constexpr (OPS > 0)
    for (uint32_t k = threadIdx.x * 16u; k < a.img_bytes; k += kThreads * 16u) *(u32x4*)(lds + a.img + k) = u32x4{0u, 0u, 0u, 0u};
  wait_tile_loads();

  // A wave takes one leaf over the tile, or over a half or quarter of it so
  // that the four waves share the leaves evenly; the leaves of the same
  // records are in work at the same time, so that their parts of one line
  // of a record-major destination meet in L2.
  const uint32_t parts = (a.nleaf & 3u) == 0u ? 1u : (a.nleaf & 1u) == 0u ? 2u : 4u;
  const uint32_t per = (nt + parts * kStep - 1u) / (parts * kStep) * kStep;
  uint32_t f = wave_id(), r0 = 0;
  for (;; f += nw) {
    while (f >= a.nleaf) {
      f -= a.nleaf;
      r0 += per;
    }
    if (r0 >= nt) break;
    const uint32_t r1 = r0 + per < nt ? r0 + per : nt;
    const TreeLeaf lf = a.leaf[f];
    uint8_t* base = a.dleaf[f];
    Place sp{lf.steps & 0xFFFFu, 0u, 0u, {}}, dp{lf.steps >> 16, 0u, 0u, {}};
    if (((lf.src | lf.dst) >> 28) & 1u) {
      const TreeGroup &sg = a.sg[(lf.src >> 25) & 7u], &dg = a.dg[(lf.dst >> 25) & 7u];
      if ((lf.src >> 28) & 1u) sp.L = sg.L, sp.block = sg.block, sp.div_L = sg.div_L;
      if ((lf.dst >> 28) & 1u) dp.L = dg.L, dp.block = dg.block, dp.div_L = dg.div_L, base += (uint64_t)t * dg.tstride;
      else base += i0 * dp.step;
      tree_leaf<OPS, true>(a, lf, sp, dp, base, lds, r0, r1);
    } else {
      tree_leaf<OPS, false>(a, lf, sp, dp, base + i0 * dp.step, lds, r0, r1);
    }
  }
  if (a.images == 0u) return;  // uniform
  __syncthreads();
  // the images, 1 KiB groups of all of them in turn
  turn = wave_id();
  auto store_image = [&](const uint8_t* img, uint8_t* out, uint32_t bytes) {
    const uint32_t groups = (bytes + 1023u) >> 10;
    uint32_t grp = turn;
    for (; grp < groups; grp += nw) {
      const uint32_t b = grp * 1024u + lane * 16u;
      if (b + 16u <= bytes) {
        __builtin_nontemporal_store(*(const u32x4*)(img + b), (u32x4*)(out + b));
      } else {
        for (uint32_t k = b; k < bytes; ++k) out[k] = img[k];
      }
    }
    turn = grp - groups;
  };
  for (uint32_t g = 0; g < kMaxGroups; ++g) {
    const TreeGroup& dg = a.dg[g];
    if (dg.image) store_image(lds + (dg.image & 0xFFFFu), a.dcol[dg.image >> 16] + (uint64_t)t * dg.tstride, nt * dg.block);
  }
  if constexpr (OPS > 0) {
    if (a.img_bytes == 0u) return;
    for (uint32_t q = 0; q < a.nleaf; ++q) {
      const TreeLeaf lf = a.leaf[q];
      const uint32_t bits = (lf.dst >> 4) & 127u;
      if ((lf.dst & 3u) == TR_BITS)  // whole words: the bits past the last code are 0
        store_image(lds + (lf.lds >> 16), a.dleaf[q] + (i0 >> 3) * bits, ((nt * bits + 31u) >> 5) * 4u);
    }
  }
}

hipError_t launch_tree(const TreeArgs& a, uint32_t ops, uint32_t grid, uint32_t lds, hipStream_t st) {
  switch (ops) {
    case 0: hipLaunchKernelGGL(k_tree<0>, dim3(grid), dim3(kThreads), lds, st, a); break;
    case 1: hipLaunchKernelGGL(k_tree<1>, dim3(grid), dim3(kThreads), lds, st, a); break;
    default: hipLaunchKernelGGL(k_tree<2>, dim3(grid), dim3(kThreads), lds, st, a); break;
  }
  return hipGetLastError();
}

}  // namespace lm
