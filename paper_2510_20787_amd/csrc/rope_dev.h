// Inverse rotary embedding of cached keys on the device (paper Section 3.1.3, lazy scoring paragraph: the cache holds
// the keys after the rotation, the scoring CNN wants them as they were before it, so they are rotated back with the
// model's cached sinusoids and negated sines).  Shared by the batched scoring of the decode ring and by the
// continuation of a prefill.
#pragma once
#include "ltea_common.h"

namespace ltea {

struct RopeDev {
  const float *cos, *sin;   // [n_pos][rot_dim / 2]
  int n_pos, rot_dim, interleaved;
};

inline RopeDev rope_dev(const ltea_rope* rope) {
  return RopeDev{rope ? rope->cos : nullptr, rope ? rope->sin : nullptr, rope ? rope->n_pos : 0,
                 rope ? rope->rot_dim : 0, rope ? rope->interleaved : 0};
}

template <typename T> struct Elems;   // 16 bytes <-> fp32 values
template <> struct Elems<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void unpack(const u32x4& r, float (&x)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(r[i]);
  }
  static __device__ __forceinline__ u32x4 pack(const float (&x)[4]) {
    return u32x4{__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3])};
  }
};
template <> struct Elems<bf16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void unpack(const u32x4& r, float (&x)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = __uint_as_float(r[i] << 16);
      x[2 * i + 1] = __uint_as_float(r[i] & 0xFFFF0000u);
    }
  }
  static __device__ __forceinline__ u32x4 pack(const float (&x)[8]) {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      r[i] = (uint32_t)__builtin_bit_cast(uint16_t, from_f32<bf16_t>(x[2 * i])) |
             ((uint32_t)__builtin_bit_cast(uint16_t, from_f32<bf16_t>(x[2 * i + 1])) << 16);
    return r;
  }
};

// The table entries of the piece at element e0 (below rot_dim) of a key at position p (below n_pos): one per element, or, in
// the interleaved order, one per pair in the first half.  16-byte loads where the tables are only known to be 4-byte aligned.
template <typename T> struct RopeEntries { float c[Elems<T>::N], s[Elems<T>::N]; };
template <typename T>
__device__ __forceinline__ RopeEntries<T> load_rope_entries(const RopeDev& rope, int p, int e0) {
  constexpr int EPP = Elems<T>::N;
  const int half = rope.rot_dim / 2;
  typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
  typedef float f32x2_any __attribute__((ext_vector_type(2), aligned(4)));
  RopeEntries<T> E;
  if (rope.interleaved) {
    const float *ct = rope.cos + (int64_t)p * half + e0 / 2, *st = rope.sin + (int64_t)p * half + e0 / 2;
#pragma unroll
    for (int j = 0; j < EPP / 2; j += 2) {
      const f32x2_any c2 = *reinterpret_cast<const f32x2_any*>(ct + j), s2 = *reinterpret_cast<const f32x2_any*>(st + j);
      E.c[j] = c2[0]; E.c[j + 1] = c2[1]; E.s[j] = s2[0]; E.s[j + 1] = s2[1];
    }
#pragma unroll
    for (int j = EPP / 2; j < EPP; ++j) E.c[j] = E.s[j] = 0.f;
  } else {
    const int i0 = e0 >= half ? e0 - half : e0;
    const float *ct = rope.cos + (int64_t)p * half + i0, *st = rope.sin + (int64_t)p * half + i0;
#pragma unroll
    for (int j = 0; j < EPP; j += 4) {
      const f32x4_any c4 = *reinterpret_cast<const f32x4_any*>(ct + j), s4 = *reinterpret_cast<const f32x4_any*>(st + j);
#pragma unroll
      for (int i = 0; i < 4; ++i) { E.c[j + i] = c4[i]; E.s[j + i] = s4[i]; }
    }
  }
  return E;
}

// First element of the piece that holds the other members of this piece's pairs (the piece itself in the interleaved order).
__device__ __forceinline__ int rope_partner(const RopeDev& rope, int e0) {
  const int half = rope.rot_dim / 2;
  return rope.interleaved ? e0 : e0 >= half ? e0 - half : e0 + half;
}

// The piece at element e0, rotated back and rounded to the storage type.  Inverse rotation of the pair (a, b):
// (a cos + b sin, -a sin + b cos).
template <typename T>
__device__ __forceinline__ u32x4 rotate_back(const RopeDev& rope, int e0, const RopeEntries<T>& E, const u32x4& piece,
                                             const u32x4& partner) {
  constexpr int EPP = Elems<T>::N;
  float x[EPP], y[EPP];
  Elems<T>::unpack(piece, x);
  if (rope.interleaved) {
#pragma unroll
    for (int j = 0; j < EPP; j += 2) {
      const float c = E.c[j / 2], s = E.s[j / 2];
      y[j] = fmaf(x[j + 1], s, x[j] * c);
      y[j + 1] = fmaf(x[j + 1], c, -(x[j] * s));
    }
  } else {
    const bool is_b = e0 >= rope.rot_dim / 2;           // this piece holds the second members of its pairs
    float o[EPP];
    Elems<T>::unpack(partner, o);
#pragma unroll
    for (int j = 0; j < EPP; ++j) y[j] = is_b ? fmaf(x[j], E.c[j], -(o[j] * E.s[j])) : fmaf(o[j], E.s[j], x[j] * E.c[j]);
  }
  return Elems<T>::pack(y);
}

// The 16-byte piece starting at element e0 of the key row `row` (the row as cached, i.e. rotated at position p),
// rotated back and rounded to the storage type.  `piece` is that piece as already loaded.  Elements at or beyond
// rot_dim pass through.  The caller has checked p < rope.n_pos.
template <typename T>
__device__ __forceinline__ u32x4 unrotate_piece(const RopeDev& rope, int p, int e0, const u32x4& piece, const T* row) {
  if (e0 >= rope.rot_dim) return piece;
  const RopeEntries<T> E = load_rope_entries<T>(rope, p, e0);
  const u32x4 other = rope.interleaved ? piece : *reinterpret_cast<const u32x4*>(row + rope_partner(rope, e0));
  return rotate_back<T>(rope, e0, E, piece, other);
}

}  // namespace ltea
