// Value-level copies: dst(i).f = src(i).f with each value loaded through the
// source mapping and stored through the destination mapping (Sec. 1 copy;
// Sec. 3 computed mappings), for the pairs the tile kernels do not move:
// two computed views (bit-packed to bit-packed, ChangeType to ChangeType with
// conversions on both sides), integer ChangeType, bit-packed codes of 33 to
// 64 bits, bit-packed floats of f16 / bf16 leaves, SPLIT trees with computed
// parts against a partner of another form; of those, the pairs that the tiled
// form (k_tree.hip) leaves: sides in different linearisation orders, AoSoA
// blocks that fit no tile or only a few long ones.  One thread takes 32
// consecutive records (of the destination's order) and moves them field by
// field: 32 codes of B bits are exactly B whole stream words, so a bit-packed
// destination is written without atomics, one word at a time as the codes
// fill it.
#include "mixing.hpp"
#include "value_codec.hpp"

namespace lm {

// B bits at stream bit `bit` (B <= 64: at most three words)
__device__ __forceinline__ uint64_t gen_read_bits(const uint8_t* stream, uint64_t bit, uint32_t B) {
  const uint32_t* w = (const uint32_t*)stream + (bit >> 5);
  const uint32_t sh = (uint32_t)(bit & 31u);
  const uint32_t nw = (sh + B + 31u) >> 5;
  unsigned __int128 acc = 0;
  for (uint32_t k = 0; k < nw; ++k) acc |= (unsigned __int128)w[k] << (32u * k);
  return (uint64_t)(acc >> sh) & low_mask64(B);
}

__device__ __forceinline__ uint64_t gen_load(const GenSide& s, const GenArgs& a, uint64_t i, uint32_t f) {
  const uint32_t ut = a.user_t[f];
  switch (s.kind[f]) {
    case GK_NULL: return 0ull;
    case GK_PHYS: return mix_load(s.m, i, f, (uint32_t)__builtin_ctz(gen_bytes(ut)));
    case GK_CONV: {
      const uint32_t st = s.stored_t[f];
      return gen_convert(mix_load(s.m, i, f, (uint32_t)__builtin_ctz(gen_bytes(st))), st, ut);
    }
    case GK_BITS_INT: {
      const uint32_t B = s.bits[f];
      const uint64_t c = gen_read_bits(s.m.col[s.m.cidx[f]], i * B, B);
      uint64_t v = c;
      if (gen_signed(ut) && B < 64u && ((c >> (B - 1u)) & 1ull)) v |= ~low_mask64(B);
      return v & low_mask64(8u * gen_bytes(ut));
    }
    default: {  // GK_BITS_FLOAT
      const uint32_t B = s.bits[f];
      const uint64_t c = gen_read_bits(s.m.col[s.m.cidx[f]], i * B, B);
      uint32_t Et, Mt;
      gen_float_fmt(ut, Et, Mt);
      return gen_widen(c, s.E[f], s.M[f], Et, Mt, false);
    }
  }
}

__device__ __forceinline__ uint64_t gen_encode(const GenSide& d, const GenArgs& a, uint64_t v, uint32_t f) {
  if (d.kind[f] == GK_BITS_INT) return v & low_mask64(d.bits[f]);
  uint32_t Et, Mt;
  gen_float_fmt(a.user_t[f], Et, Mt);
  return gen_narrow(v, Et, Mt, d.E[f], d.M[f], d.rne[f] != 0u);
}

__device__ __forceinline__ void gen_store(const GenSide& d, const GenArgs& a, uint64_t i, uint32_t f, uint64_t v) {
  const uint32_t ut = a.user_t[f];
  if (d.kind[f] == GK_PHYS) {
    mix_store(d.m, i, f, (uint32_t)__builtin_ctz(gen_bytes(ut)), v);
  } else {  // GK_CONV
    const uint32_t st = d.stored_t[f];
    mix_store(d.m, i, f, (uint32_t)__builtin_ctz(gen_bytes(st)), gen_convert(v, ut, st));
  }
}

__global__ __launch_bounds__(kThreads) void k_generic(GenArgs a) {
  const uint64_t groups = (a.n + 31u) >> 5;
  const uint64_t stride = (uint64_t)gridDim.x * kThreads;
  for (uint64_t g = (uint64_t)blockIdx.x * kThreads + threadIdx.x; g < groups; g += stride) {
    const uint64_t i0 = g * 32u;
    for (uint32_t f = 0; f < a.nf; ++f) {
      const uint32_t dk = a.dst.kind[f];
      if (dk == GK_NULL) continue;  // a NULL part of a SPLIT destination drops the values
      if (dk != GK_BITS_INT && dk != GK_BITS_FLOAT) {
        for (uint32_t k = 0; k < 32u && i0 + k < a.n; ++k) {
          const uint64_t i = i0 + k;
          gen_store(a.dst, a, i, f, gen_load(a.src, a, mix_src_index(a.order, i), f));
        }
        continue;
      }
      // 32 codes of B bits: the B words from word g * B on, written as they fill
      const uint32_t B = a.dst.bits[f];
      const uint64_t nw_stream = (a.n * B + 31u) >> 5;
      uint32_t* out = (uint32_t*)a.dst.m.col[a.dst.m.cidx[f]] + g * B;
      unsigned __int128 acc = 0;
      uint32_t have = 0, w = 0;
      for (uint32_t k = 0; k < 32u; ++k) {
        const uint64_t i = i0 + k;
        const uint64_t c = i < a.n ? gen_encode(a.dst, a, gen_load(a.src, a, mix_src_index(a.order, i), f), f) : 0ull;
        acc |= (unsigned __int128)c << have;
        have += B;
        while (have >= 32u) {
          if (g * B + w < nw_stream) out[w] = (uint32_t)acc;
          acc >>= 32;
          have -= 32u;
          ++w;
        }
      }
    }
  }
}

hipError_t launch_generic(const GenArgs& a, uint32_t grid, hipStream_t st) {
  hipLaunchKernelGGL(k_generic, dim3(grid), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace lm
