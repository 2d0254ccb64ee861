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
