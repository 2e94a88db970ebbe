/* Stands in for the library in tests/test_binding.py: every function writes down its arguments. */
#include "shiftattn.h"
static struct { const void *p[9]; int32_t i[7]; float f; size_t n; int which; } seen;
const void *stub_seen(void) { return &seen; }
size_t stub_size(void) { return sizeof seen; }
#define CLEAR(w) do { char *c = (char *)&seen; for (size_t k = 0; k < sizeof seen; ++k) c[k] = 0; seen.which = w; } while (0)
#define P(k, v) seen.p[k] = (const void *)(v)
int sp_kv_append(const sp_cache_desc *cache, const void *k, const void *v, const int32_t *cu, const int32_t *ctx, const int32_t *bt,
                 int32_t a, int32_t b, int32_t c, void *s) {
  CLEAR(1); P(0, cache->k_pages); P(1, k); P(2, v); P(3, cu); P(4, ctx); P(5, bt); P(8, s);
  seen.i[0] = a; seen.i[1] = b; seen.i[2] = c; seen.i[6] = cache->num_pages; return 0;
}
int sp_attn_prefill(const sp_cache_desc *cache, const void *q, void *out, const int32_t *cu, const int32_t *ctx, const int32_t *bt, int32_t a,
                    int32_t b, int32_t c, int32_t d, int32_t e, int32_t f, float scale, int32_t causal, void *ws, size_t n, void *s) {
  CLEAR(2); P(0, cache->k_pages); P(1, q); P(2, out); P(3, cu); P(4, ctx); P(5, bt); P(7, ws); P(8, s);
  seen.i[0] = a; seen.i[1] = b; seen.i[2] = c; seen.i[3] = d; seen.i[4] = e; seen.i[5] = f; seen.i[6] = causal; seen.f = scale; seen.n = n;
  return -2;
}
int sp_chunk_step(const sp_cache_desc *cache, const void *k, const void *v, const void *q, void *out, const int32_t *cu, const int32_t *ctx,
                  const int32_t *bt, int32_t a, int32_t b, int32_t c, int32_t d, int32_t e, int32_t f, float scale, void *ws, size_t n, void *s) {
  CLEAR(3); P(0, k); P(1, v); P(2, q); P(3, out); P(4, cu); P(5, ctx); P(6, bt); P(7, ws); P(8, s);
  seen.i[0] = a; seen.i[1] = b; seen.i[2] = c; seen.i[3] = d; seen.i[4] = e; seen.i[5] = f; seen.i[6] = cache->num_pages; seen.f = scale; seen.n = n;
  return 0;
}
int sp_attn_decode(const sp_cache_desc *cache, const void *q, void *out, const int32_t *lens, const int32_t *bt, int32_t a, int32_t b, int32_t c,
                   int32_t d, float scale, void *ws, size_t n, void *s) {
  CLEAR(4); P(0, cache->k_pages); P(1, q); P(2, out); P(3, lens); P(4, bt); P(7, ws); P(8, s);
  seen.i[0] = a; seen.i[1] = b; seen.i[2] = c; seen.i[3] = d; seen.f = scale; seen.n = n; return -4;
}
int sp_attn_decode_static(const sp_cache_desc *cache, const void *q, void *out, const int32_t *lens, const int32_t *bt, int32_t a, int32_t b,
                          int32_t c, int32_t d, float scale, void *s) {
  CLEAR(5); P(0, cache->k_pages); P(1, q); P(2, out); P(3, lens); P(4, bt); P(8, s);
  seen.i[0] = a; seen.i[1] = b; seen.i[2] = c; seen.i[3] = d; seen.f = scale; return 0;
}
int sp_decode_step(const sp_cache_desc *cache, const void *k, const void *v, const void *q, void *out, const int32_t *lens, const int32_t *bt,
                   int32_t a, int32_t b, int32_t c, int32_t d, float scale, void *ws, size_t n, void *s) {
  CLEAR(6); P(0, cache->v_pages); P(1, k); P(2, v); P(3, q); P(4, out); P(5, lens); P(6, bt); P(7, ws); P(8, s);
  seen.i[0] = a; seen.i[1] = b; seen.i[2] = c; seen.i[3] = d; seen.f = scale; seen.n = n; return 0;
}
