// The UTF-8 reading of word bytes: one byte at a time from any source, and 16 bytes per lane.
#pragma once

#include "wc_internal.h"

namespace wc {

// ---- UTF-8 tokeniser (the "other languages" of Section 5.2) ---------------------------------
// A byte is a word byte when it belongs to a well-formed UTF-8 sequence (Unicode Standard,
// Table 3-7) that lies inside one document and whose code point is a word character: the
// ASCII word bytes, or any code point from U+0080 up except U+0080..U+00BF, U+00D7, U+00F7,
// U+2000..U+206F, U+3000..U+303F and U+FEFF. Folding stays ASCII-only.
WC_DEV bool utf8_word_cp(uint32_t cp) {
  if (cp <= 0xBF || cp == 0xD7 || cp == 0xF7 || cp == 0xFEFF) return false;
  if (cp >= 0x2000 && cp <= 0x206F) return false;
  if (cp >= 0x3000 && cp <= 0x303F) return false;
  return true;
}

// Sequence length (2..4) of a lead byte c, the allowed range of the byte after it and the
// lead's code point bits; 0 when c does not start a multi-byte sequence.
WC_DEV uint32_t utf8_lead(uint32_t c, uint32_t* lo2, uint32_t* hi2, uint32_t* v) {
  *lo2 = 0x80u;
  *hi2 = 0xBFu;
  if (c >= 0xC2u && c <= 0xDFu) {
    *v = c & 0x1Fu;
    return 2;
  }
  if (c >= 0xE0u && c <= 0xEFu) {
    *v = c & 0x0Fu;
    if (c == 0xE0u) *lo2 = 0xA0u;
    if (c == 0xEDu) *hi2 = 0x9Fu;
    return 3;
  }
  if (c >= 0xF0u && c <= 0xF4u) {
    *v = c & 0x07u;
    if (c == 0xF0u) *lo2 = 0x90u;
    if (c == 0xF4u) *hi2 = 0x8Fu;
    return 4;
  }
  return 0;
}

// Word flag of the byte at logical position q under the UTF-8 reading. Bytes exist in
// [lo, hi); byte_at(x) reads one, starts_at(x) tells whether a document starts at x (a
// sequence never spans a document start).
template <class ByteAt, class StartsAt>
WC_DEV uint32_t utf8_word_byte(int64_t q, int64_t lo, int64_t hi, ByteAt byte_at,
                               StartsAt starts_at) {
  if (q < lo || q >= hi) return 0u;
  uint32_t c = byte_at(q);
  if (c < 0x80u) return is_word_byte(c) ? 1u : 0u;
  int64_t j = q;
  for (int k = 0; c >= 0x80u && c <= 0xBFu; ++k) {  // a continuation: step back to its lead
    if (k == 3 || j == lo || starts_at(j)) return 0u;
    c = byte_at(--j);
  }
  uint32_t lo2, hi2, v;
  const uint32_t n = utf8_lead(c, &lo2, &hi2, &v);
  if (n == 0 || j + (int64_t)n <= q) return 0u;
  for (uint32_t t = 1; t < n; ++t) {
    const int64_t x = j + t;
    if (x >= hi || starts_at(x)) return 0u;
    const uint32_t d = byte_at(x);
    if (d < (t == 1 ? lo2 : 0x80u) || d > (t == 1 ? hi2 : 0xBFu)) return 0u;
    v = (v << 6) | (d & 0x3Fu);
  }
  return utf8_word_cp(v) ? 1u : 0u;
}

// A document starts at logical position q (some offsets[d] == q, 1 <= d <= n_docs).
WC_DEV bool doc_starts_at(const uint64_t* offsets, uint64_t n_docs, int64_t q) {
  uint64_t a = 1, b = n_docs + 1;
  while (a < b) {
    const uint64_t m = (a + b) >> 1;
    if ((int64_t)offsets[m] < q) a = m + 1;
    else b = m;
  }
  return a <= n_docs && (int64_t)offsets[a] == q;
}

// Word bytes among the multi-byte sequences that start in 16 bytes g (ASCII folded): bit j for byte
// j, bits 16..18 for the bytes after them. next: the four bytes after g; starts: bit j set when
// a document starts at byte j (a sequence holds no document start but at its first byte). One
// iteration per lead byte of the lane with the most; lanes without one cost nothing.
WC_DEV uint32_t utf8_mask(const uint4 g, uint32_t next, uint32_t starts) {
  const uint32_t H = 0x80808080u;  // leads have the two top bits set
  uint32_t leads = movemask16(g.x & (g.x << 1) & H, g.y & (g.y << 1) & H, g.z & (g.z << 1) & H,
                              g.w & (g.w << 1) & H);
  uint32_t res = 0;
  while (leads) {
    const uint32_t j = __ffs(leads) - 1, k = j >> 2;
    leads &= leads - 1;
    const uint32_t a = k == 0 ? g.x : k == 1 ? g.y : k == 2 ? g.z : g.w;
    const uint32_t b = k == 0 ? g.y : k == 1 ? g.z : k == 2 ? g.w : next;
    const uint32_t w = __builtin_amdgcn_alignbyte(b, a, j & 3);
    const uint32_t c0 = w & 0xffu, c1 = (w >> 8) & 0xffu;
    uint32_t lo2, hi2, v;
    const uint32_t n = utf8_lead(c0, &lo2, &hi2, &v);
    if (n == 0) continue;
    const uint32_t tail = n == 2 ? 0x0000ff00u : n == 3 ? 0x00ffff00u : 0xffffff00u;
    const bool cont = ((w ^ 0x80808080u) & 0xc0c0c0c0u & tail) == 0;
    const bool whole = (starts & (((1u << n) - 2u) << j)) == 0;
    v = (v << 6) | (c1 & 0x3fu);
    if (n > 2) v = (v << 6) | ((w >> 16) & 0x3fu);
    if (n > 3) v = (v << 6) | ((w >> 24) & 0x3fu);
    if (cont && whole && c1 >= lo2 && c1 <= hi2 && utf8_word_cp(v)) res |= ((1u << n) - 1u) << j;
  }
  return res;
}

}  // namespace wc
