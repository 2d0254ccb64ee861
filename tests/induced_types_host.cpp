// Host build of the text functions of cxbwt_induce.h for a CPU test: suffix
// types, preceding bases and later windows, the code the kernels run.
#include "cxbwt_induce.h"

extern "C" void it_type(const void *text, uint64_t p, uint32_t *out) {
  const cxk::TextRec *t = static_cast<const cxk::TextRec *>(text);
  const SuffixType ty = suffix_type(t, t[p >> 4], p);
  out[0] = ty.base;
  out[1] = ty.run;
  out[2] = ty.s;
  out[3] = base_before(t[p >> 4], (uint32_t)(p & 15));
}
extern "C" uint32_t it_preceding(const void *text, uint64_t p, int end) {
  return preceding(static_cast<const cxk::TextRec *>(text), p, end != 0);
}
extern "C" uint32_t it_trim(uint32_t pl) { return pl_trim(pl); }
extern "C" uint32_t it_run(uint32_t pl) { return pl_run(pl); }
extern "C" uint64_t it_window(const void *text, uint64_t q, uint32_t full, uint32_t *clamp) {
  return later_window(static_cast<const cxk::TextRec *>(text)[q >> 4], q, full, *clamp);
}
// The samples of a record's positions in [a, e), bit o for position 16 w + o;
// bit 16: the record takes the slow way.
extern "C" uint32_t it_samples(const void *text, uint64_t w, uint64_t a, uint64_t e) {
  const cxk::TextRec *t = static_cast<const cxk::TextRec *>(text);
  const uint32_t valid = lanes_within(w, a, e);
  const RecordTypes ty = record_types(t[w]);
  const uint32_t m = ty.slow ? slow_samples(t, t[w], w, valid) : ty.sample & valid;
  uint32_t r = ty.slow ? 1u << 16 : 0u;
  for (uint32_t o = 0; o < 16; ++o) r |= ((m >> (30 - 2 * o)) & 1u) << o;
  return r;
}
// S-type positions and positions equal to the next, the same way.
extern "C" void it_masks(const void *text, uint64_t w, uint32_t *out) {
  const RecordTypes ty = record_types(static_cast<const cxk::TextRec *>(text)[w]);
  out[0] = out[1] = 0;
  for (uint32_t o = 0; o < 16; ++o) {
    out[0] |= ((ty.s >> (30 - 2 * o)) & 1u) << o;
    out[1] |= ((ty.eq >> (30 - 2 * o)) & 1u) << o;
  }
}
