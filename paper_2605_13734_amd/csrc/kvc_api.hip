// Host side of the C ABI (include/kvc.h): plan validation, payload geometry and header,
// and the launch sequences of kvc_compress / kvc_decompress.  No device allocation, no
// synchronisation; everything is enqueued on the caller's stream.

#include <stdlib.h>
#include <string.h>

#include <mutex>

#include "../../include/kvc.h"
#include "kvc_internal.h"

using namespace kvc;

struct kvc_plan_s {
    kvc_model model;
    kvc_strategy strat;
    int64_t max_tokens;
    int32_t max_batch;
    size_t ws_request;          // workspace bytes per request
    size_t ws_state_off;        // offset of the scan state inside a request's workspace
    // per-head bit widths (section 5.1: head-wise mixed precision; the MixHQ mechanism)
    int has_table[2];           // K, V
    uint8_t *blob;              // host image of the device tables, see table_layout
    size_t blob_bytes;          // multiple of 256; the workspace starts with a copy of it
    int width_count[2][4];      // heads per width 2, 3, 4, 8
    // measurement hook (kvc_trace): events recorded between the stages of a call
    hipEvent_t *trace;
    int trace_cap, trace_n;
};

static const int kWidths[4] = {2, 3, 4, 8};
// limits that keep every byte count of a payload below 2^63
static const long long kMaxHeads = 1ll << 20, kMaxTokens = 1ll << 32;

// Device tables of a plan with per-head widths, in this order (LH = layers * kv_heads):
//   aux image : the bytes of the payload's auxiliary section (K table, V table, zero padding
//               to 16 bytes)
//   per tensor: long long bits_before[LH], then int head_list[LH] (heads grouped by width, in
//               the order 2, 3, 4, 8; head order kept inside a group)
struct TableLayout {
    size_t aux_image, bits_before[2], head_list[2], total;
};
static TableLayout table_layout(long long LH, int tables)
{
    TableLayout t;
    size_t at = 0;
    t.aux_image = at;
    at += (size_t)((tables * LH + 15) & ~15ll);
    at = (at + 255) & ~(size_t)255;
    for (int i = 0; i < 2; ++i) {
        t.bits_before[i] = at;
        at += (size_t)LH * 8;
        t.head_list[i] = at;
        at += (((size_t)LH * 4) + 7) & ~(size_t)7;
    }
    t.total = (at + 255) & ~(size_t)255;
    return t;
}

// The coder's workspace of a request: [slots][kSampleChunks][256] byte counts, [kTableSlots][4096] table words,
// the ticket's 256 bytes, the scan state.
static int table_slots(const kvc_plan_t *p) { return (p->has_table[0] || p->has_table[1]) ? kTableSlots : 2; }
static size_t lut_offset(const kvc_plan_t *p) { return (size_t)table_slots(p) * kSampleChunks * 256 * 2; }
static size_t ticket_offset(const kvc_plan_t *p) { return lut_offset(p) + (size_t)kTableSlots * 4096 * 2; }

static int width_at(const kvc_plan_t *p, int is_v, long long lh)
{
    const uint8_t *t = is_v ? p->strat.head_bits_v : p->strat.head_bits_k;
    return t ? t[lh] : (is_v ? p->strat.bits_v : p->strat.bits_k);
}

// Optional measurement hook (kvc_trace): events recorded between the stages of a call, four per
// request: before anything of the request is enqueued, after its set-up, after K, after V.  Requests
// that share their launches (see request_window) share the moments.
struct Marks {
    kvc_plan_t *p;
    hipStream_t s;
    int base;
    Marks(const kvc_plan_t *plan, hipStream_t stream) : p(const_cast<kvc_plan_t *>(plan)), s(stream), base(p->trace_n) {}
    void at(int request, int stage) const
    {
        const int idx = base + 4 * request + stage;
        if (p->trace && idx < p->trace_cap && hipEventRecord(p->trace[idx], s) == hipSuccess && p->trace_n < idx + 1) p->trace_n = idx + 1;
    }
    void window(int first, int end, int stage) const
    {
        if (!p->trace) return;
        for (int i = first; i < end; ++i)
            if (!(stage == 0 && i == 0)) at(i, stage);      // (the first request's first mark opens the call)
    }
};

extern "C" int kvc_trace(kvc_plan_t *plan, void **hip_events, int32_t capacity)
{
    if (!plan) return 0;
    const int recorded = plan->trace_n;
    plan->trace = (hipEvent_t *)hip_events;
    plan->trace_cap = hip_events ? capacity : 0;
    plan->trace_n = 0;
    return recorded;
}

static inline long long a16(long long n) { return (n + 15) & ~15ll; }
static inline size_t a256(size_t n) { return (n + 255) & ~(size_t)255; }

static bool bits_ok(int b) { return b == 2 || b == 3 || b == 4 || b == 8 || b == 16; }
static bool group_ok(int g) { return g == 32 || g == 64 || g == 128; }

static long long chunks_per_head(long long tokens) { return (tokens + kChunkRows - 1) / kChunkRows; }

// Payload = header | K meta | V meta | auxiliary section | K codes | V codes, each part on a
// 16-byte boundary; two fp16 values of metadata per group (section 7.3).  The auxiliary section
// holds the coder's tables and directory or the per-head width tables, then (delta transform, from
// the next 16-byte boundary) the anchor rows of K and of V, 16 bits per element.
static long long anchor_rows(const kvc_plan_t *p, int is_v, long long T)
{
    if (p->strat.transform != KVC_T_DELTA) return 0;
    if (!p->has_table[is_v] && (is_v ? p->strat.bits_v : p->strat.bits_k) == 16) return 0;
    return (T + p->strat.anchor_period - 1) / p->strat.anchor_period;
}

static void geometry(const kvc_plan_t *p, long long T, Geometry *g)
{
    const long long LH = (long long)p->model.layers * p->model.kv_heads, D = p->model.head_dim;
    const int bk = p->strat.bits_k, bv = p->strat.bits_v;
    g->meta_k = (bk == 16 && !p->has_table[0]) ? 0 : 4 * LH * ((T + p->strat.group_k - 1) / p->strat.group_k) * D;
    g->meta_v = (bv == 16 && !p->has_table[1]) ? 0 : 4 * LH * T * (D / p->strat.group_v);
    long long sum_k = LH * bk, sum_v = LH * bv;          // widths summed over the heads
    if (p->has_table[0]) {
        sum_k = 0;
        for (long long i = 0; p->strat.head_bits_k && i < LH; ++i) sum_k += p->strat.head_bits_k[i];
    }
    if (p->has_table[1]) {
        sum_v = 0;
        for (long long i = 0; p->strat.head_bits_v && i < LH; ++i) sum_v += p->strat.head_bits_v[i];
    }
    g->codes_k = sum_k * T * D / 8;
    g->codes_v = sum_v * T * D / 8;
    g->chunks_k = g->chunks_v = LH * chunks_per_head(T);
    // with the coder: its tables (one per tensor, or one per tensor and width when there are width
    // tables), then the directory; then the width tables
    g->code_tables = p->strat.codec ? 256 * ((p->has_table[0] || p->has_table[1]) ? kTableSlots : 2) : 0;
    g->aux = p->strat.codec ? g->code_tables + 4 * (g->chunks_k + g->chunks_v + 1) : 0;
    g->widths = (p->has_table[0] + p->has_table[1]) * LH;
    const long long widths_at = g->aux;
    g->aux += g->widths;
    g->aux_base = g->aux;
    g->anchors_k = 2 * LH * anchor_rows(p, 0, T) * D;
    g->anchors_v = 2 * LH * anchor_rows(p, 1, T) * D;
    if (p->strat.transform == KVC_T_DELTA) g->aux = a16(g->aux_base) + g->anchors_k + g->anchors_v;
    g->off_meta_k = kHeader;
    g->off_meta_v = g->off_meta_k + a16(g->meta_k);
    g->off_aux = g->off_meta_v + a16(g->meta_v);
    g->off_dir = g->off_aux + g->code_tables;
    g->off_widths = g->off_aux + widths_at;
    g->off_codes_k = g->off_aux + a16(g->aux);
    g->off_anchors_k = g->off_codes_k - g->anchors_v - g->anchors_k;
    g->off_anchors_v = g->off_codes_k - g->anchors_v;
    g->off_codes_v = g->off_codes_k + a16(g->codes_k);
    g->total = g->off_codes_v + a16(g->codes_v);
}

static void put16(uint8_t *p, unsigned v) { p[0] = (uint8_t)v; p[1] = (uint8_t)(v >> 8); }
static void put32(uint8_t *p, uint32_t v) { for (int i = 0; i < 4; ++i) p[i] = (uint8_t)(v >> (8 * i)); }
static void put64(uint8_t *p, uint64_t v) { for (int i = 0; i < 8; ++i) p[i] = (uint8_t)(v >> (8 * i)); }
static unsigned get16(const uint8_t *p) { return p[0] | (p[1] << 8); }
static uint32_t get32(const uint8_t *p) { uint32_t v = 0; for (int i = 0; i < 4; ++i) v |= (uint32_t)p[i] << (8 * i); return v; }
static uint64_t get64(const uint8_t *p) { uint64_t v = 0; for (int i = 0; i < 8; ++i) v |= (uint64_t)p[i] << (8 * i); return v; }

// 128-byte little-endian header.  With the coder, the four size-dependent fields (total,
// K code bytes, V code offset, V code bytes) are left zero here and patched on the device.
static void make_header(const kvc_plan_t *p, long long T, const Geometry &g, HeaderBytes *out)
{
    uint8_t h[kHeader];
    memset(h, 0, sizeof h);
    memcpy(h, "KVC1", 4);
    put16(h + 4, 1);
    h[6] = p->model.dtype;
    h[7] = p->strat.codec;
    put32(h + 8, (uint32_t)p->model.layers);
    put32(h + 12, (uint32_t)p->model.kv_heads);
    put32(h + 16, (uint32_t)p->model.head_dim);
    h[20] = p->has_table[0] ? 0 : p->strat.bits_k;
    h[21] = p->has_table[1] ? 0 : p->strat.bits_v;
    put16(h + 22, p->strat.group_k);
    put16(h + 24, p->strat.group_v);
    h[26] = p->strat.transform;
    h[27] = (uint8_t)(p->has_table[0] | (p->has_table[1] << 1));
    put16(h + 28, p->strat.anchor_period);
    put64(h + 32, (uint64_t)T);
    put64(h + 48, (uint64_t)g.off_meta_k); put64(h + 56, (uint64_t)g.meta_k);
    put64(h + 64, (uint64_t)g.off_meta_v); put64(h + 72, (uint64_t)g.meta_v);
    put64(h + 80, (uint64_t)g.off_aux);    put64(h + 88, (uint64_t)g.aux);
    put64(h + 96, (uint64_t)g.off_codes_k);
    if (!p->strat.codec) {
        put64(h + 40, (uint64_t)g.total);
        put64(h + 104, (uint64_t)g.codes_k);
        put64(h + 112, (uint64_t)g.off_codes_v);
        put64(h + 120, (uint64_t)g.codes_v);
    }
    memcpy(out->w, h, kHeader);
}

extern "C" const char *kvc_status_string(int s)
{
    switch (s) {
    case KVC_OK: return "ok";
    case KVC_ERR_ARG: return "invalid argument";
    case KVC_ERR_UNSUPPORTED: return "unsupported configuration";
    case KVC_ERR_CAPACITY: return "capacity too small";
    case KVC_ERR_FORMAT: return "malformed payload";
    case KVC_ERR_MISMATCH: return "payload does not match plan";
    case KVC_ERR_DEVICE: return "HIP error";
    }
    return "unknown status";
}

static int check_pair(const kvc_model *m, const kvc_strategy *s)
{
    if (!m || !s) return KVC_ERR_ARG;
    if (m->dtype != KVC_F16 && m->dtype != KVC_BF16) return KVC_ERR_ARG;
    if (m->layers < 1 || m->kv_heads < 1 || m->head_dim < 1) return KVC_ERR_ARG;
    if ((long long)m->layers * m->kv_heads > kMaxHeads) return KVC_ERR_ARG;      // sizes stay far below 2^63
    if ((!s->head_bits_k && !bits_ok(s->bits_k)) || (!s->head_bits_v && !bits_ok(s->bits_v))) return KVC_ERR_ARG;
    if (s->codec != KVC_CODEC_NONE && s->codec != KVC_CODEC_HUFF8) return KVC_ERR_ARG;
    if ((s->head_bits_k || s->bits_k != 16) && !group_ok(s->group_k)) return KVC_ERR_ARG;
    if ((s->head_bits_v || s->bits_v != 16) && !group_ok(s->group_v)) return KVC_ERR_ARG;
    const long long LH = (long long)m->layers * m->kv_heads;
    for (int is_v = 0; is_v < 2; ++is_v) {
        const uint8_t *t = is_v ? s->head_bits_v : s->head_bits_k;
        if (!t) continue;
        if ((is_v ? s->bits_v : s->bits_k) != 0) return KVC_ERR_ARG;        // the table replaces the uniform width
        for (long long i = 0; i < LH; ++i)
            if (t[i] != 2 && t[i] != 3 && t[i] != 4 && t[i] != 8) return KVC_ERR_ARG;
    }
    if (m->head_dim != kDim) return KVC_ERR_UNSUPPORTED;
    if (s->transform > KVC_T_DELTA) return KVC_ERR_UNSUPPORTED;
    if (s->transform == KVC_T_DELTA) {
        const int a = s->anchor_period;
        if (a < 8 || a > 128 || (a & (a - 1))) return KVC_ERR_ARG;
    } else if (s->anchor_period != 0) return KVC_ERR_ARG;
    if (s->codec && (s->bits_k == 16 || s->bits_v == 16)) return KVC_ERR_UNSUPPORTED;
    return KVC_OK;
}

extern "C" int kvc_plan(const kvc_model *model, const kvc_strategy *strategy, int64_t max_tokens,
                        int32_t max_batch, kvc_plan_t **out)
{
    if (!out) return KVC_ERR_ARG;
    *out = nullptr;
    int rc = check_pair(model, strategy);
    if (rc) return rc;
    if (max_tokens < 0 || max_tokens > kMaxTokens || max_batch < 1) return KVC_ERR_ARG;
    kvc_plan_t *p = (kvc_plan_t *)calloc(1, sizeof(kvc_plan_t));
    if (!p) return KVC_ERR_ARG;
    p->model = *model;
    p->strat = *strategy;
    if (p->strat.bits_k == 16) p->strat.group_k = 32;       // unused; keep the header canonical
    if (p->strat.bits_v == 16) p->strat.group_v = 32;
    p->max_tokens = max_tokens;
    p->max_batch = max_batch;
    p->has_table[0] = strategy->head_bits_k ? 1 : 0;
    p->has_table[1] = strategy->head_bits_v ? 1 : 0;
    p->strat.head_bits_k = p->strat.head_bits_v = nullptr;
    if (p->has_table[0] || p->has_table[1]) {
        // the plan owns copies of the tables, inside the image of the device tables
        const long long LH = (long long)model->layers * model->kv_heads;
        const TableLayout t = table_layout(LH, p->has_table[0] + p->has_table[1]);
        p->blob = (uint8_t *)calloc(1, t.total);
        if (!p->blob) { free(p); return KVC_ERR_ARG; }
        p->blob_bytes = t.total;
        uint8_t *aux = p->blob + t.aux_image;
        if (p->has_table[0]) { memcpy(aux, strategy->head_bits_k, (size_t)LH); p->strat.head_bits_k = aux; aux += LH; }
        if (p->has_table[1]) { memcpy(aux, strategy->head_bits_v, (size_t)LH); p->strat.head_bits_v = aux; }
        for (int is_v = 0; is_v < 2; ++is_v) {
            if (!p->has_table[is_v]) continue;
            long long *before = (long long *)(p->blob + t.bits_before[is_v]);
            int *list = (int *)(p->blob + t.head_list[is_v]);
            long long sum = 0, at = 0;
            for (long long i = 0; i < LH; ++i) { before[i] = sum; sum += width_at(p, is_v, i); }
            for (int w = 0; w < 4; ++w) {
                p->width_count[is_v][w] = 0;
                for (long long i = 0; i < LH; ++i)
                    if (width_at(p, is_v, i) == kWidths[w]) { list[at++] = (int)i; ++p->width_count[is_v][w]; }
            }
        }
    }
    if (strategy->codec) {
        // byte counts of the sample, code / decode tables, ticket, then the scan state:
        // one scan-state word per chunk of K and of V
        const long long chunks = (long long)model->layers * model->kv_heads * chunks_per_head(max_tokens);
        p->ws_state_off = ticket_offset(p) + 256;
        p->ws_request = p->ws_state_off + a256((size_t)(2 * chunks) * 8 + 8);
    }
    *out = p;
    return KVC_OK;
}

extern "C" void kvc_plan_free(kvc_plan_t *plan)
{
    if (plan) free(plan->blob);
    free(plan);
}

extern "C" int kvc_payload_size(const kvc_plan_t *plan, int64_t tokens, uint64_t *bytes, int *is_exact)
{
    if (!plan || !bytes || tokens < 0 || tokens > kMaxTokens) return KVC_ERR_ARG;
    Geometry g;
    geometry(plan, tokens, &g);
    *bytes = (uint64_t)g.total;
    if (is_exact) *is_exact = plan->strat.codec == 0;
    return KVC_OK;
}

extern "C" size_t kvc_workspace_size(const kvc_plan_t *plan)
{
    return plan ? plan->blob_bytes + plan->ws_request * (size_t)plan->max_batch : 0;
}

extern "C" int kvc_payload_inspect(const void *header128, kvc_model *model, kvc_strategy *strategy,
                                   int64_t *tokens, uint64_t *total_bytes, uint64_t *sections)
{
    const uint8_t *h = (const uint8_t *)header128;
    if (!h) return KVC_ERR_ARG;
    if (memcmp(h, "KVC1", 4) != 0 || get16(h + 4) != 1) return KVC_ERR_FORMAT;
    kvc_model m;
    kvc_strategy s;
    memset(&m, 0, sizeof m);
    memset(&s, 0, sizeof s);
    m.dtype = h[6];
    s.codec = h[7];
    m.layers = (int32_t)get32(h + 8);
    m.kv_heads = (int32_t)get32(h + 12);
    m.head_dim = (int32_t)get32(h + 16);
    s.bits_k = h[20];
    s.bits_v = h[21];
    s.group_k = (uint16_t)get16(h + 22);
    s.group_v = (uint16_t)get16(h + 24);
    s.transform = h[26];
    s.anchor_period = (uint16_t)get16(h + 28);
    const int64_t T = (int64_t)get64(h + 32);
    // a tensor with a per-head width table has width 0 in the header; the table itself is in the
    // auxiliary section, which this function does not see
    const int flags = h[27];
    if (flags & ~3) return KVC_ERR_FORMAT;
    kvc_strategy probe = s;
    if (flags & 1) { if (s.bits_k) return KVC_ERR_FORMAT; probe.bits_k = 4; }
    if (flags & 2) { if (s.bits_v) return KVC_ERR_FORMAT; probe.bits_v = 4; }
    int rc = check_pair(&m, &probe);
    if (rc == KVC_ERR_ARG || T < 0 || T > kMaxTokens) return KVC_ERR_FORMAT;
    if (h[30] | h[31]) return KVC_ERR_FORMAT;
    // the fixed part of the section table must be the closed form of the fields above
    kvc_plan_t tmp;
    memset(&tmp, 0, sizeof tmp);
    tmp.model = m;
    tmp.strat = s;
    tmp.has_table[0] = flags & 1;
    tmp.has_table[1] = (flags >> 1) & 1;
    Geometry g;
    geometry(&tmp, T, &g);
    const uint64_t want[7] = {(uint64_t)g.off_meta_k, (uint64_t)g.meta_k, (uint64_t)g.off_meta_v,
                              (uint64_t)g.meta_v, (uint64_t)g.off_aux, (uint64_t)g.aux,
                              (uint64_t)g.off_codes_k};
    for (int i = 0; i < 7; ++i)
        if (get64(h + 48 + 8 * i) != want[i]) return KVC_ERR_FORMAT;
    const uint64_t total = get64(h + 40), ck = get64(h + 104), ov = get64(h + 112), cv = get64(h + 120);
    // with width tables the code sizes follow from the tables, which are not in the header: only the
    // bounds that hold for any table (2 to 8 bits per element) are known here
    const uint64_t unit = (uint64_t)m.layers * m.kv_heads * (uint64_t)T * 16;      // bytes per bit of width
    const uint64_t lo_k = (flags & 1) ? 2 * unit : (uint64_t)s.bits_k * unit, hi_k = (flags & 1) ? 8 * unit : lo_k;
    const uint64_t lo_v = (flags & 2) ? 2 * unit : (uint64_t)s.bits_v * unit, hi_v = (flags & 2) ? 8 * unit : lo_v;
    if (flags && s.codec) {
        if (ov != (uint64_t)g.off_codes_k + ck || total != ov + cv || (ck & 15) || (cv & 15) || ck > hi_k || cv > hi_v)
            return KVC_ERR_FORMAT;
    } else if (flags) {
        if (ck < lo_k || ck > hi_k || cv < lo_v || cv > hi_v || ov != (uint64_t)g.off_codes_k + (uint64_t)a16((long long)ck) ||
            total != ov + (uint64_t)a16((long long)cv))
            return KVC_ERR_FORMAT;
    } else if (!s.codec) {
        if (total != (uint64_t)g.total || ck != (uint64_t)g.codes_k || ov != (uint64_t)g.off_codes_v ||
            cv != (uint64_t)g.codes_v)
            return KVC_ERR_FORMAT;
    } else {
        if (ov != (uint64_t)g.off_codes_k + ck || total != ov + cv || total > (uint64_t)g.total ||
            (ck & 15) || (cv & 15))
            return KVC_ERR_FORMAT;
    }
    if (model) *model = m;
    if (strategy) *strategy = s;
    if (tokens) *tokens = T;
    if (total_bytes) *total_bytes = total;
    if (sections) {
        for (int i = 0; i < 7; ++i) sections[i] = want[i];
        sections[7] = ck; sections[8] = ov; sections[9] = cv;
    }
    return rc;     // KVC_OK, or KVC_ERR_UNSUPPORTED for a well-formed header this build cannot run
}

extern "C" int kvc_check_block_table(const int32_t *table, int64_t entries, int32_t num_phys_blocks)
{
    if (!table || entries < 0 || num_phys_blocks < 1) return KVC_ERR_ARG;
    for (int64_t i = 0; i < entries; ++i)
        if (table[i] < 0 || table[i] >= num_phys_blocks) return KVC_ERR_ARG;
    return KVC_OK;
}

static bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

static int check_request(const kvc_plan_t *p, const kvc_request *r)
{
    if (r->tokens < 0) return KVC_ERR_ARG;
    if (r->tokens > p->max_tokens) return KVC_ERR_CAPACITY;
    if (r->tokens == 0) return KVC_OK;
    if (!r->k || !r->v || !aligned16(r->k) || !aligned16(r->v)) return KVC_ERR_ARG;
    if ((r->stride_layer | r->stride_head | r->stride_token) & 7) return KVC_ERR_ARG;
    if (r->stride_token < kDim) return KVC_ERR_ARG;
    if (r->block_table) {
        if (r->block_tokens < 1 || (r->block_tokens & (r->block_tokens - 1))) return KVC_ERR_UNSUPPORTED;
        if (r->num_phys_blocks < 1 || (r->stride_block & 7) || r->stride_block < 1) return KVC_ERR_ARG;
        if (((uintptr_t)r->block_table & 3)) return KVC_ERR_ARG;
    }
    return KVC_OK;
}

static TensorView view_of(const kvc_request *r, int is_v)
{
    TensorView v;
    v.base = (uint16_t *)(is_v ? r->v : r->k);
    v.stride_layer = r->stride_layer;
    v.stride_head = r->stride_head;
    v.stride_token = r->stride_token;
    v.stride_block = r->stride_block;
    v.block_table = r->block_table;
    v.bt_shift = 0;
    if (r->block_table)
        while ((1 << v.bt_shift) < r->block_tokens) ++v.bt_shift;
    v.num_phys_blocks = r->num_phys_blocks;
    v.bt_wave = (r->block_table && r->block_tokens >= 4 && r->stride_token < (1ll << 24) &&
                 (long long)r->block_tokens * r->stride_token < (1ll << 31)) ? 1 : 0;
    return v;
}

static QuantArgs quant_args(const kvc_plan_t *p, const kvc_request *r, int is_v, uint8_t *payload,
                            const Geometry &g, int *status, bool compress)
{
    QuantArgs a;
    memset(&a, 0, sizeof a);
    const int bits = is_v ? p->strat.bits_v : p->strat.bits_k;
    const int group = is_v ? p->strat.group_v : p->strat.group_k;
    a.x = view_of(r, is_v);
    a.codes = payload + (is_v ? g.off_codes_v : g.off_codes_k);
    a.meta = payload + (is_v ? g.off_meta_v : g.off_meta_k);
    a.tokens = r->tokens;
    a.heads = p->model.kv_heads;
    a.group = group;
    a.dense = (!r->block_table && r->stride_token == kDim) ? 1 : 0;
    a.head_minor = (r->stride_head < r->stride_token && !p->has_table[is_v]) ? 1 : 0;
    a.rotate = (p->strat.transform == KVC_T_HADAMARD && bits != 16) ? 1 : 0;
    if (anchor_rows(p, is_v, r->tokens) > 0) {
        a.anchors = (uint16_t *)(payload + (is_v ? g.off_anchors_v : g.off_anchors_k));
        while ((1 << a.anchor_shift) < p->strat.anchor_period) ++a.anchor_shift;
    }
    const long long rows_per_unit = (compress && !is_v && bits != 16) ? group : kPassRows;
    a.units_per_head = (r->tokens + rows_per_unit - 1) / rows_per_unit;
    a.total_units = a.units_per_head * p->model.layers * p->model.kv_heads;
    a.status = status;
    return a;
}

// One tensor of the requests of a window without the coder: one launch, or one per width present in
// the head table.
static int launch_tensor(const kvc_plan_t *p, int is_v, bool compress, QuantBatch b, const uint8_t *dev_tables, hipStream_t s)
{
    const int dt = p->model.dtype;
    const int group = is_v ? p->strat.group_v : p->strat.group_k;
    if (!p->has_table[is_v]) {
        const int bits = is_v ? p->strat.bits_v : p->strat.bits_k;
        return compress ? launch_compress_tensor(is_v, bits, group, dt, b, s) : launch_decompress_tensor(is_v, bits, group, dt, b, s);
    }
    const long long LH = (long long)p->model.layers * p->model.kv_heads;
    const TableLayout t = table_layout(LH, p->has_table[0] + p->has_table[1]);
    const int *list = (const int *)(dev_tables + t.head_list[is_v]);
    for (int w = 0; w < 4; ++w) {
        const int n = p->width_count[is_v][w];
        if (n > 0) {
            for (int i = 0; i < b.n; ++i) {
                b.item[i].bits_before = (const long long *)(dev_tables + t.bits_before[is_v]);
                b.item[i].head_list = list;
                b.item[i].total_units = b.item[i].units_per_head * n;
            }
            const int rc = compress ? launch_compress_tensor(is_v, kWidths[w], group, dt, b, s)
                                    : launch_decompress_tensor(is_v, kWidths[w], group, dt, b, s);
            if (rc) return rc;
        }
        list += n;
    }
    return KVC_OK;
}

// The requests [first, end) that share their launches: at most `limit`, of one layout class (the
// kernels for rows that are contiguous per head are not the ones for strided or paged rows), and
// small ones only -- a request that fills the chip many times over gains nothing from company, and
// finding its item costs every workgroup of a shared launch a look at the batch (measured: a batch of
// four 20k- to 30k-token requests ran 4 % slower shared than one after the other).  Empty requests
// have no work in any launch and fit every window.

// Requests of a coder window where K and V share a launch, but for wide windows.
static const int kSharedWindow = 4;

static bool dense_layout(const kvc_request *r) { return !r->block_table && r->stride_token == kDim; }

static const long long kSmallRows = 1ll << 21;           // token rows per tensor: 64 Ki work units of 32 rows

static int request_window(const kvc_plan_t *p, const kvc_request *reqs, int n, int first, int limit, int *lead)
{
    const long long heads = (long long)p->model.layers * p->model.kv_heads;
    int end = first, leader = -1;
    while (end < n && end - first < limit) {
        if (reqs[end].tokens > 0) {
            const bool small = heads * reqs[end].tokens < kSmallRows;
            if (leader < 0) leader = end;
            else if (!small || heads * reqs[leader].tokens >= kSmallRows ||
                     dense_layout(&reqs[end]) != dense_layout(&reqs[leader])) break;
        }
        ++end;
    }
    *lead = leader < 0 ? first : leader;
    return end;
}

// the k-th request of a window in launch order: the leader (a request that has rows) first, because
// the launchers read the kernel variant off the first item, then the others in their order
static int window_item(int first, int end, int lead, int k)
{
    (void)end;
    if (k == 0) return lead;
    return first + k - 1 < lead ? first + k - 1 : first + k;
}

// the window's tensor as one batch
static QuantBatch quant_batch(const kvc_plan_t *plan, const kvc_request *reqs, int first, int end, int lead, int is_v,
                              void *payload, const uint64_t *payload_off, int32_t *dev_status, bool compress)
{
    QuantBatch b;
    memset(&b, 0, sizeof b);
    for (int k = 0; k < end - first; ++k) {
        const int i = window_item(first, end, lead, k);
        Geometry g;
        geometry(plan, reqs[i].tokens, &g);
        b.item[b.n++] = quant_args(plan, &reqs[i], is_v, (uint8_t *)payload + payload_off[i], g, dev_status + i, compress);
    }
    return b;
}

extern "C" size_t kvc_table_bytes(const kvc_plan_t *plan) { return plan ? plan->blob_bytes : 0; }

extern "C" int kvc_workspace_init(const kvc_plan_t *plan, void *workspace, void *hip_stream)
{
    if (!plan) return KVC_ERR_ARG;
    if (!plan->blob_bytes) return KVC_OK;
    if (!workspace || ((uintptr_t)workspace & 15)) return KVC_ERR_ARG;
    return hipMemcpyAsync(workspace, plan->blob, plan->blob_bytes, hipMemcpyHostToDevice, (hipStream_t)hip_stream) == hipSuccess
               ? KVC_OK : KVC_ERR_DEVICE;
}

// The coder launches of a request, the same for all requests of a plan, in chunk order: K before V; a tensor with a width table
// is one launch per width present (2, 3, 4, 8) over the heads of that width, otherwise one launch.
struct CoderLaunch {
    int is_v, bits, group, tab;
    int heads;                  // heads it covers
    const int *head_list;       // ... (null without a width table: the heads in their own order)
};
struct CoderLaunches {
    CoderLaunch of[kTableSlots];
    int n, slots;               // CoderArgs::slots
};

// Whether K and V of the requests of a window share a launch with the coder.  The kernels for both tensors
// exist for one width and one group for both and no transform, and a shared launch takes half as many
// requests.  It pays where the two passes would leave the chip idle: one layer of 32k tokens and 8 heads: encoding
// 56 us in two launches, 45 in one, decoding 50 and 37; 2^21 rows (fp16, 4 bits): compress call 319 and
// 280 us; requests of 2^23 rows and more gain 2 % and keep their passes apart.
// - More than four requests: eight of them, K and V apart, take as many launches with twice the work in
//   each (time apart / shared, fp16, 4 bits, 5 to 8 requests of 2^14, 2^16, 2^18 and 2^19 rows each: groups of 32 1.00 0.99
//   0.95 1.01, of 64 1.00 0.92 0.95 1.00, of 128 0.99 0.95 0.89 0.89).  8-bit codes share four at a time (groups of 128, six
//   requests of 2^16 rows 1.07, others 1.00 to 1.04).
// - Groups of 64 and 128: a K kernel needs more registers than a V kernel, and in a shared launch V has the
//   waves of K.  Groups of 64 (three waves per SIMD) lose nothing by it below 2^21 rows (apart / shared, one request: 2^18 1.05,
//   2^20 1.21, 2^21 1.12).  Groups of 128 (two) do with more than 2^20 rows in the window (2^16 1.43, 2^18 0.95 to
//   0.99, 2^19 1.04 to 1.12, 2^20 1.02 to 1.10, 2^20.6 0.96 to 1.03, 2^21 0.93 to 0.98), but for 8 bits, where LDS bounds
//   the waves of either (2^21 1.10).  The strided bf16 kernel at groups of 128 has one wave per SIMD: shared only
//   while all chunks are resident at once (2^16 1.40, 2^17 0.87, 2^20 0.75, 2^21 0.72).
static bool tensors_share(const kvc_plan_t *p)
{
    const kvc_strategy &st = p->strat;
    return !p->has_table[0] && !p->has_table[1] && st.bits_k == st.bits_v && st.group_k == st.group_v && st.transform == KVC_T_NONE;
}

static const int kUnits = 256;                       // compute units

// chunks of K and V of a window; *largest: of its largest request
static long long window_chunks(const kvc_plan_t *p, const kvc_request *reqs, int first, int end, long long *largest)
{
    long long chunks = 0;
    *largest = 0;
    for (int i = first; i < end; ++i) {
        const long long c = 2ll * p->model.layers * p->model.kv_heads * chunks_per_head(reqs[i].tokens);
        chunks += c;
        *largest = c > *largest ? c : *largest;
    }
    return chunks;
}

// Whether the windows of a call are as wide as the coder's batches: from five requests on, where they have 2^21 rows per tensor together.
// Every launch less saves a start and a tail.  Time with wide windows / with windows of four (K and V together), eight and twelve
// (apart), the least and the most of 2, 3, 4 and 8 bits, K 4 and V 2, rotation and half of the heads at 8 bits, fp16 and bf16:
//   requests      5 to 8, 2^21 to 2^23 rows        9 to 16, 2^21.5 to 2^24.2    20 to 40, 2^21.5 to 2^25.1
//   compression   0.89 to 1.00 (rotation, paged 1.02)  0.86 to 0.99             0.73 to 0.99
//   decompression 0.91 to 1.01                     0.86 to 1.00                 0.76 to 0.99
// (calls with fewer rows have the windows below, whose lines were measured with batches of twelve)
static bool wide_window(const kvc_plan_t *p, const kvc_request *reqs, int n)
{
    long long per_head = 0;
    for (int i = 0; i < n; ++i) per_head += chunks_per_head(reqs[i].tokens);
    return n > kSharedWindow && per_head * p->model.layers * p->model.kv_heads >= kSmallRows / kChunkRows;
}

// Requests of a coder window where K and V share a launch (coder_window: where they go apart).
static int shared_window(const kvc_plan_t *p, const kvc_request *reqs, int n) { return wide_window(p, reqs, n) ? kCoderBatch / 2 : kSharedWindow; }

// Requests of a coder window with K and V apart: eight, from seventeen on twelve.  A window is a start and a tail per launch, but
// where a launch of twelve of the widest codes has up to a quarter more chunks than are resident (16 per compute unit, at 8 bits 8; with width
// tables, whose launches are smaller, up to a half) its rest has the chip to itself, and eight is better unless twelve takes a
// window less for every such rest.  Time with twelve / with eight, 17, 24 and 32 requests, 64 heads of 400 to 2100 tokens each or 8
// and 256 heads of 300 to 2000, fp16 and bf16:
//   where twelve is taken   compression 0.70 to 0.99, decompression 0.56 to 1.00 (K 4 and V 2 bits, a rest of a third or half 1.02 to 1.04)
//   where eight is taken    compression, half of the heads at 8 bits 1.01 to 1.05, rotation and 8 bits 1.09, 4 bits 1.02 (2 bits groups
//                           of 128, rotation and 4 bits 0.94 to 0.98); decompression, K 4 and V 2 bits 1.06 to 1.10, 8 bits 1.14
//   sixteen requests take two windows either way: 12 + 4 against 8 + 8 0.82 to 1.17
// (Nine to twelve requests would gain by one window, 0.58 to 0.97, but for 1.03 at one size; they take eight and the rest.)
static int coder_window(const kvc_plan_t *p, const kvc_request *reqs, int n)
{
    const int most = 12;
    if (wide_window(p, reqs, n)) return kCoderBatch;
    if (n <= 16) return 8;
    if (2 * (n / most) + (n % most > 0) <= (n + 7) / 8) return most;
    long long per_head = 0, heads[2] = {0, 0};
    for (int i = 0; i < n; ++i) per_head += chunks_per_head(reqs[i].tokens);
    int widest = 0;
    for (int w = 0; w < 4; ++w) {
        long long has[2];
        for (int is_v = 0; is_v < 2; ++is_v)
            has[is_v] = p->has_table[is_v] ? p->width_count[is_v][w]
                        : kWidths[w] == (is_v ? p->strat.bits_v : p->strat.bits_k) ? (long long)p->model.layers * p->model.kv_heads : 0;
        if (has[0] + has[1] == 0) continue;
        widest = kWidths[w];
        heads[0] = has[0];
        heads[1] = has[1];
    }
    const long long resident = (widest == 8 ? 8ll : 16ll) * kUnits * n;                  // (times n, as the chunks)
    for (int is_v = 0; is_v < 2; ++is_v) {
        const long long chunks = heads[is_v] * per_head * most;
        if (chunks > resident && 4 * chunks <= (p->has_table[is_v] ? 6 : 5) * resident) return 8;
    }
    return most;
}

static bool share_kv(const kvc_plan_t *p, const kvc_request *reqs, int first, int end, int lead, int limit)
{
    if (!tensors_share(p) || end - first > limit) return false;
    const long long rows = (long long)p->model.layers * p->model.kv_heads * reqs[lead].tokens;
    if (p->strat.group_k == 32) return rows < 4 * kSmallRows;
    if (rows >= kSmallRows) return false;
    long long largest;
    const long long chunks = window_chunks(p, reqs, first, end, &largest);
    // (more than four requests of groups of 64: shared up to 3 * 2^21 rows 0.93 to 0.98 of the time apart, above 1.01 to 1.02)
    if (p->strat.group_k == 64) return end - first <= kSharedWindow || chunks <= 6 * kSmallRows / kChunkRows;
    if (p->model.dtype == KVC_BF16 && !dense_layout(&reqs[lead])) return chunks <= 4 * kUnits;
    return p->strat.bits_k == 8 || chunks <= kSmallRows / kChunkRows;        // 2^20 rows of K and of V
}

// The decoder has no order to keep and takes the group as a run-time value, so there K and V share a launch for
// every width that both have: also with different groups, and with width tables (half of the heads at
// 8 bits, half at 2, 2^21 rows: decompress call 411 us with K and V apart, 367 together).
// Of the widths that K or V have: 2 if both have all of them, 1 some, 0 none (or a transform).
static int common_widths(const kvc_plan_t *p)
{
    int any = 0, both = 0;
    for (int w = 0; w < 4; ++w) {
        int has = 0;
        for (int is_v = 0; is_v < 2; ++is_v)
            has += p->has_table[is_v] ? p->width_count[is_v][w] > 0 : kWidths[w] == (is_v ? p->strat.bits_v : p->strat.bits_k);
        any += has > 0;
        both += has == 2;
    }
    if (both == 0 || p->strat.transform != KVC_T_NONE) return 0;
    return both == any ? 2 : 1;
}

// A shared launch takes four requests, in a wide window sixteen.  Where both tensors have all widths, two windows of four take as many
// launches as one of eight with K and V apart; where one of them has a width of its own they take more, and of the windows that are not
// wide those of more than four requests stay apart (K 4 and 3 bits, V 4 and 2, five requests of 2^14, 2^16 and 2^18 rows:
// 66 81 208 us apart, 88 100 203 shared; K 8, 4 and 2 bits, V 8 and 2: 106 120 304 and 125 139 291).  Wide ones share (256 heads, apart /
// shared: K 4 and 3, V 4 and 2 bits, 5 requests of up to 2048 tokens 309 / 291 us, 8 of 1100 279 / 262, 16 of 1800 842 / 822; K 8, 4 and 2, V
// 8 and 2 394 / 369, 363 / 332, 1081 / 1080).
static bool widths_share(const kvc_plan_t *p, const kvc_request *reqs, int first, int end, int lead, int limit)
{
    return common_widths(p) > 0 && end - first <= limit &&
           (long long)p->model.layers * p->model.kv_heads * reqs[lead].tokens < 4 * kSmallRows;
}

// Chunks per workgroup of an encoder launch for both tensors (0: the usual number), where all chunks of
// the window are resident at once (16 waves per compute unit) and the usual number would queue for more than 256
// tickets, which are one after the other (one layer as above: 72 us per call with four, 66 with eight).  With
// more work the tickets hide behind other workgroups and four wait less for each other (enc_waves).  Between 8
// and 12 waves per unit three workgroups of four share the work evenly, where some units have two of eight and
// others one (2432 chunks of four requests 59 us with eight, 53 with four); a single request's tickets cost more than
// that from 10 waves per unit up (2816 chunks, 2 bits, 53.5 and 54.6, 3072 54.5 and 57.0; 4 bits level).
static int shared_waves(const kvc_plan_t *p, const kvc_request *reqs, int first, int end)
{
    if (p->strat.group_k != 32 || p->strat.bits_k == 8) return 0;
    long long largest;
    const long long chunks = window_chunks(p, reqs, first, end, &largest);
    if (chunks <= 4 * kUnits || chunks > 16 * kUnits) return 0;
    return chunks > 8 * kUnits && chunks <= 12 * kUnits && largest <= 10 * kUnits ? 0 : 8;
}

static CoderLaunches coder_launches(const kvc_plan_t *p, const uint8_t *dev_tables)
{
    const bool any_table = table_slots(p) == kTableSlots;
    const long long LH = (long long)p->model.layers * p->model.kv_heads;
    const TableLayout t = table_layout(LH, p->has_table[0] + p->has_table[1]);
    CoderLaunches all;
    memset(&all, 0, sizeof all);
    all.slots = table_slots(p) << 8;
    for (int is_v = 0; is_v < 2; ++is_v) {
        const int *list = p->has_table[is_v] ? (const int *)(dev_tables + t.head_list[is_v]) : nullptr;
        for (int w = 0; w < 4; ++w) {
            long long heads = 0;
            if (p->has_table[is_v]) heads = p->width_count[is_v][w];
            else if (kWidths[w] == (is_v ? p->strat.bits_v : p->strat.bits_k)) heads = LH;
            if (heads == 0) continue;
            CoderLaunch &l = all.of[all.n++];
            l.is_v = is_v;
            l.bits = kWidths[w];
            l.group = is_v ? p->strat.group_v : p->strat.group_k;
            l.tab = any_table ? 4 * is_v + w : is_v;
            l.heads = (int)heads;
            l.head_list = list;
            if (list) list += heads;
            all.slots |= 1 << l.tab;
        }
    }
    return all;
}

// encode workgroups of all launches of a request; *k_wgs: of its K launches.  waves: chunks per workgroup (0: enc_waves)
static long long encode_workgroups(const CoderLaunches &all, long long tokens, int waves, long long *k_wgs)
{
    long long wgs = 0;
    *k_wgs = 0;
    for (int j = 0; j < all.n; ++j) {
        const int nw = waves ? waves : enc_waves(all.of[j].bits);
        wgs += (all.of[j].heads * chunks_per_head(tokens) + nw - 1) / nw;
        if (!all.of[j].is_v) *k_wgs = wgs;
    }
    return wgs;
}

// The items of a request, `number` behind the window's first, for all launches.
static void coder_items(const kvc_plan_t *p, const CoderLaunches &all, const kvc_request *r, uint8_t *payload, long long capacity, int number,
                        int waves, CoderItem out[kTableSlots])
{
    Geometry g;
    geometry(p, r->tokens, &g);
    const QuantArgs q[2] = {quant_args(p, r, 0, payload, g, nullptr, true), quant_args(p, r, 1, payload, g, nullptr, true)};
    long long k_wgs, chunk_at = 0, wg_at = 0;
    const long long total_wgs = encode_workgroups(all, r->tokens, waves, &k_wgs);
    for (int j = 0; j < all.n; ++j) {
        const CoderLaunch &l = all.of[j];
        CoderItem &it = out[j];
        const TensorView &x = q[l.is_v].x;
        it.base = x.base;
        it.stride_layer = x.stride_layer;
        it.stride_head = x.stride_head;
        it.stride_token = x.stride_token;
        it.stride_block = x.stride_block;
        it.block_table = x.block_table;
        it.num_phys_blocks = x.num_phys_blocks;
        it.payload = payload;
        it.capacity = capacity;
        it.tokens = r->tokens;
        const long long places[4] = {l.is_v ? g.off_meta_v : g.off_meta_k, g.off_aux, g.off_codes_k,
                                     !q[l.is_v].anchors ? 0 : l.is_v ? g.off_anchors_v : g.off_anchors_k};
        it.off_meta = (uint32_t)(places[0] / 16);
        it.off_aux = (uint32_t)(places[1] / 16);
        it.off_bodies = (uint32_t)(places[2] / 16);
        it.off_anchors = (uint32_t)(places[3] / 16);
        it.chunk_base = (uint32_t)chunk_at;
        it.wg_base = (uint32_t)wg_at;
        it.k_wgs = (uint32_t)k_wgs;
        it.total_wgs = (uint32_t)total_wgs;
        it.flags = (uint32_t)(x.bt_shift | x.bt_wave << 5 | q[l.is_v].head_minor << 6 | l.is_v << 7 | l.tab << 8 | number << 11);
        for (int k = 0; k < 4; ++k) it.flags |= (uint32_t)(places[k] >> 36) << (16 + 4 * k);
        const int nw = waves ? waves : enc_waves(l.bits);
        const long long chunks = l.heads * chunks_per_head(r->tokens);
        chunk_at += chunks;
        wg_at += (chunks + nw - 1) / nw;
    }
}

static void add_item(CoderBatch &b, const CoderLaunch &l, const CoderItem &it)
{
    b.item[b.n++] = it;
    b.head_list[l.is_v] = l.head_list;
    b.heads_covered[l.is_v] = l.heads;
    b.group[l.is_v] = l.group;
}

// Whether the workgroups that build the code tables of a window's requests have no chunks of their own.  They are better apart: the
// scan starts at the first tickets, and those who build have their chunks late.  But where the window's first launch is resident at
// once and with them it would not be, as many workgroups would start when the first of the others end.  Compress call, fp16, 4
// bits, groups of 32, with chunks / apart (in a launch of their own before): one request of 8 heads, 30000 tokens 55.2 / 51.7 us, 32768
// (exactly resident) 57.4 / 68.1 (66.1), 36000 76.8 / 72.7; four of 8192 56.6 / 63.5, of 24000 132.7 / 122.7; 8 bits, 12288 tokens 58.9 /
// 53.7, 16384 64.2 / 74.9, 20000 85.3 / 80.3; groups of 128, 16384 tokens 45.3 / 54.1, 32768 79.1 / 74.9; half of the heads at 2 bits,
// half at 8, 64 heads of 8192 166.9 / 162.3.  (32 requests of 256 heads and 512 to 2048 tokens, in windows of twelve, 1448 / 1348 (1365).)
// first: the window's first launch; how many of its workgroups are resident the runtime knows, by kernel.  kv, dtype: of that launch
static bool builders_apart(const CoderBatch &first, const CoderLaunch &l, int kv, int dtype, int builders)
{
    const int nw = first.waves ? first.waves : enc_waves(l.bits);
    long long wgs = 0;
    for (int i = 0; i < first.n; i += kv == 2 ? 2 : 1) {
        const long long w = kv == 2 ? (long long)first.item[i].total_wgs : (item_chunks(first, i) + nw - 1) / nw;
        if (w < builders) return true;                   // (not enough of them)
        wgs += w;
    }
    int resident = 0;
    if (launch_encode_section(kv, l.bits, l.group, dtype, first, nullptr, &resident) != KVC_OK) return true;
    return wgs > resident || wgs + (long long)(kv == 2 ? first.n / 2 : first.n) * builders <= resident;
}

// A batch without items for a window from request `first` on whose rows lie as those of `lead` do.
static CoderBatch coder_batch(const kvc_plan_t *p, const CoderLaunches &all, const kvc_request *lead, int first, void *workspace, uint64_t *out_bytes,
                              int *status)
{
    CoderBatch b;
    memset(&b, 0, sizeof b);
    b.ws_request = (long long)p->ws_request;
    b.ws = (uint8_t *)workspace + p->blob_bytes + first * b.ws_request;
    b.status = status + first;
    b.out_bytes = out_bytes ? (unsigned long long *)out_bytes + first : nullptr;
    b.ws_lut = (uint32_t)lut_offset(p);
    b.ws_ticket = (uint32_t)ticket_offset(p);
    b.ws_state = (uint32_t)p->ws_state_off;
    b.heads = p->model.kv_heads;
    b.all_heads = p->model.layers * p->model.kv_heads;
    b.dense = dense_layout(lead) ? 1 : 0;
    b.rotate = p->strat.transform == KVC_T_HADAMARD ? 1 : 0;
    while ((1 << b.anchor_shift) < p->strat.anchor_period) ++b.anchor_shift;
    b.slots = all.slots;
    return b;
}

// Whether the coder's items can hold the places of a request (CoderItem).  What they cannot is beyond any buffer of a GPU, and a launch
// has fewer than 2^26 chunks (2^24 workgroups of 256 threads).
static bool places_fit(const Geometry &g) { return g.off_codes_k >> 40 == 0 && (g.chunks_k + g.chunks_v) >> 31 == 0; }

static int check_batch(const kvc_plan_t *p, const kvc_request *reqs, int32_t n, const void *payload,
                       const uint64_t *off, const void *workspace)
{
    if (!p || !reqs || n < 1 || !payload || !off || !aligned16(payload)) return KVC_ERR_ARG;
    if (n > p->max_batch) return KVC_ERR_CAPACITY;
    if ((p->ws_request || p->blob_bytes) && (!workspace || !aligned16(workspace))) return KVC_ERR_ARG;
    for (int i = 0; i < n; ++i) {
        int rc = check_request(p, &reqs[i]);
        if (rc) return rc;
        if ((off[i] & 15) || off[i + 1] < off[i]) return KVC_ERR_ARG;
    }
    return KVC_OK;
}

#define KVC_TRY(expr) do { int rc__ = (expr); if (rc__ != KVC_OK) return rc__; } while (0)

// A call without the coder that fits one launch: up to four requests without a block table, of one layout
// class, K and V of one width and group, no transform and no width tables, and few enough rows that
// launches, latency and the tail of the K pass are part of what the call costs.  One launch is the
// faster one at every size below the line, in both directions, for both types, all widths and groups
// (compress / decompress call, fp16, rows per tensor, in three launches and in one: 2 bits g64 2^16 17.8 / 14.2 and 11.8 /
// 8.9 us, 2^18 39 / 31 and 31 / 26, 2^20 109 / 95 and 101 / 88, just below 2^21 213 / 182 and 210 / 177; 8 bits g32
// 17.9 / 15.5 and 11.2 / 10.0, 45 / 44 and 37 / 38, 141 / 140 and 133 / 133, 269 / 276 and 266 / 266).  Above it
// K and V of a request are long enough to be worth a mark each (kvc_trace).
static const long long kSmallCallRows = 1ll << 21;       // token rows per tensor of the whole call

static bool small_call(const kvc_plan_t *p, const kvc_request *reqs, int n)
{
    const kvc_strategy &st = p->strat;
    if (st.codec || n > kSmallRequests || !tensors_share(p) || st.bits_k == 16) return false;
    long long rows = 0;
    for (int i = 0; i < n; ++i) {
        if (reqs[i].block_table && reqs[i].tokens > 0) return false;
        if (reqs[i].tokens > 0 && reqs[0].tokens > 0 && dense_layout(&reqs[i]) != dense_layout(&reqs[0])) return false;
        rows += (long long)p->model.layers * p->model.kv_heads * reqs[i].tokens;
    }
    return reqs[0].tokens > 0 && rows < kSmallCallRows;
}

// What the prologue writes for one request (ws: its part of the coder's workspace, or null).
static void prologue_item(const kvc_plan_t *plan, const kvc_request *r, uint8_t *payload, void *workspace, uint8_t *ws,
                          uint64_t *out_bytes, int32_t *status, PrologueItem *item)
{
    Geometry g;
    geometry(plan, r->tokens, &g);
    PrologueItem &it = *item;
    it.payload = (uint32_t *)payload;
    make_header(plan, r->tokens, g, &it.header);
    // alignment padding after the V metadata and after the coder's or the width tables is zero
    it.pad_off[0] = g.off_meta_v + g.meta_v;
    it.pad_words[0] = (int)((a16(g.meta_v) - g.meta_v) / 4);
    it.pad_off[1] = g.off_aux + g.aux_base;
    it.pad_words[1] = (int)((a16(g.aux_base) - g.aux_base) / 4);
    if (plan->blob_bytes) {
        // the width tables: a copy of the image at the start of the workspace (whole words; the
        // image is zero behind the tables), then zero up to the next 16-byte boundary
        it.aux_src = (const uint32_t *)workspace;
        it.aux_off = g.off_widths;
        it.aux_words = (g.widths + 3) / 4;
        it.pad_off[1] = g.off_widths + 4 * it.aux_words;
        it.pad_words[1] = (int)((g.off_aux + a16(g.aux_base) - it.pad_off[1]) / 4);
    }
    it.out_bytes = (unsigned long long *)out_bytes;
    it.status = status;
    if (!plan->strat.codec) {
        it.total = (unsigned long long)g.total;
        it.write_total = 1;
        return;
    }
    // candidate tables, ticket and scan state start from zero
    uint32_t *ticket = (uint32_t *)(ws + ticket_offset(plan));
    long long k_wgs;
    it.zero = (uint32_t *)candidate_tables(ticket, table_slots(plan) - 1);
    it.zero_words = (ticket - it.zero) + 64 + 2 * encode_workgroups(coder_launches(plan, (const uint8_t *)workspace), r->tokens, 0, &k_wgs) + 2;
    if (r->tokens == 0) {
        // empty request: no workgroup runs that could close the directory and header
        put64((uint8_t *)it.header.w + 40, (uint64_t)g.off_codes_k);
        put64((uint8_t *)it.header.w + 112, (uint64_t)g.off_codes_k);
        it.dir0 = (uint32_t *)(payload + g.off_dir);
        it.total = (unsigned long long)g.off_codes_k;
        it.write_total = 1;
    }
}

// Set-up of all requests of a call with the coder: prologues and table samples (the first encoder launch builds the tables).
static int coder_setup(const kvc_plan_t *plan, const kvc_request *reqs, int32_t n, void *payload, const uint64_t *payload_off,
                       uint64_t *out_bytes, int32_t *dev_status, void *workspace, hipStream_t s)
{
    const kvc_strategy &st = plan->strat;
    const long long LH = (long long)plan->model.layers * plan->model.kv_heads;
    const TableLayout t = table_layout(LH, plan->has_table[0] + plan->has_table[1]);
    SetupArgs sa;
    memset(&sa, 0, sizeof sa);
    sa.heads = plan->model.kv_heads;
    const bool all_slots = table_slots(plan) == kTableSlots;
    for (int is_v = 0; is_v < 2; ++is_v) {
        const int *list = plan->has_table[is_v] ? (const int *)((const uint8_t *)workspace + t.head_list[is_v]) : nullptr;
        for (int w = 0; w < 4; ++w) {
            long long heads = 0;
            if (list) heads = plan->width_count[is_v][w];
            else if (kWidths[w] == (is_v ? st.bits_v : st.bits_k)) heads = LH;
            if (heads == 0) continue;
            SetupTable &tab = sa.table[sa.tables++];
            tab.head_list = list;
            if (list) list += heads;
            tab.heads_covered = (int)heads;
            tab.slot = all_slots ? 4 * is_v + w : is_v;
            tab.is_v = is_v;
            tab.bits = kWidths[w];
            tab.group = is_v ? st.group_v : st.group_k;
            tab.rotate = st.transform == KVC_T_HADAMARD;
            tab.anchor_shift = -1;
            if (st.transform == KVC_T_DELTA) {
                tab.anchor_shift = 0;
                while ((1 << tab.anchor_shift) < st.anchor_period) ++tab.anchor_shift;
            }
        }
    }
    for (int first = 0; first < n; first += kSetupBatch) {
        sa.n = n - first < kSetupBatch ? n - first : kSetupBatch;
        for (int j = 0; j < sa.n; ++j) {
            const int i = first + j;
            SetupItem &it = sa.item[j];
            memset(&it, 0, sizeof it);
            uint8_t *ws = (uint8_t *)workspace + plan->blob_bytes + (size_t)i * plan->ws_request;
            prologue_item(plan, &reqs[i], (uint8_t *)payload + payload_off[i], workspace, ws, out_bytes + i, dev_status + i, &it.prologue);
            it.x = view_of(&reqs[i], 0);
            it.v_base = (uint16_t *)reqs[i].v;
            it.tokens = reqs[i].tokens;
            it.sample = (uint16_t *)ws;
        }
        KVC_TRY(launch_setup(plan->model.dtype, sa, s));
    }
    return KVC_OK;
}

// The launch sequence of kvc_compress on a given workspace (the caller's, or the library's own
// static one): the set-up of all requests, then one pass per tensor over the requests of a window.
static int compress_on(const kvc_plan_t *plan, const kvc_request *reqs, int32_t n, void *payload,
                       const uint64_t *payload_off, uint64_t *out_bytes, int32_t *dev_status,
                       void *workspace, hipStream_t s)
{
    KVC_TRY(check_batch(plan, reqs, n, payload, payload_off, workspace));
    if (!out_bytes || !dev_status || ((uintptr_t)out_bytes & 7) || ((uintptr_t)dev_status & 3)) return KVC_ERR_ARG;
    for (int i = 0; i < n; ++i) {
        Geometry g;
        geometry(plan, reqs[i].tokens, &g);
        if (payload_off[i + 1] - payload_off[i] < (uint64_t)g.total) return KVC_ERR_CAPACITY;
        if (plan->strat.codec && !places_fit(g)) return KVC_ERR_UNSUPPORTED;
    }
    const kvc_strategy &st = plan->strat;
    const int dt = plan->model.dtype;
    const Marks marks(plan, s);
    marks.at(0, 0);
    marks.window(0, n, 0);                     // (the set-up of all requests comes first)
    if (small_call(plan, reqs, n)) {
        marks.window(0, n, 1);
        SmallCompressArgs sc;
        memset(&sc, 0, sizeof sc);
        for (int i = 0; i < n; ++i) {
            Geometry g;
            geometry(plan, reqs[i].tokens, &g);
            uint8_t *pl = (uint8_t *)payload + payload_off[i];
            for (int is_v = 0; is_v < 2; ++is_v) sc.item[sc.n++] = quant_args(plan, &reqs[i], is_v, pl, g, dev_status + i, true);
            prologue_item(plan, &reqs[i], pl, workspace, nullptr, out_bytes + i, dev_status + i, &sc.prologue[i]);
        }
        sc.requests = n;
        KVC_TRY(launch_compress_call(st.bits_k, st.group_k, dt, sc, s));
        marks.window(0, n, 2);
        marks.window(0, n, 3);
        return KVC_OK;
    }
    if (st.codec) {
        KVC_TRY(coder_setup(plan, reqs, n, payload, payload_off, out_bytes, dev_status, workspace, s));
    } else {
        for (int first = 0; first < n; first += kPrologueBatch) {
            PrologueArgs pa;
            memset(&pa, 0, sizeof pa);
            pa.n = n - first < kPrologueBatch ? n - first : kPrologueBatch;
            for (int j = 0; j < pa.n; ++j) {
                const int i = first + j;
                prologue_item(plan, &reqs[i], (uint8_t *)payload + payload_off[i], workspace, nullptr, out_bytes + i, dev_status + i,
                              &pa.item[j]);
            }
            KVC_TRY(launch_compress_prologue(pa, s));
        }
    }
    const int coder_limit = coder_window(plan, reqs, n), shared_limit = shared_window(plan, reqs, n);
    const CoderLaunches all = coder_launches(plan, (const uint8_t *)workspace);
    for (int first = 0; first < n;) {
        int lead;
        int end = request_window(plan, reqs, n, first, st.codec ? coder_limit : kQuantBatch, &lead);
        bool share = st.codec && share_kv(plan, reqs, first, end, lead, shared_limit);
        if (st.codec && st.bits_k == 8 && end - first > kSharedWindow && shared_limit == kSharedWindow) {
            int lead_half;
            const int half = request_window(plan, reqs, n, first, kSharedWindow, &lead_half);
            share = share_kv(plan, reqs, first, half, lead_half, shared_limit);
            if (share) {
                end = half;
                lead = lead_half;
            }
        }
        if (!st.codec) {
            marks.window(first, end, 1);
            KVC_TRY(launch_tensor(plan, 0, true, quant_batch(plan, reqs, first, end, lead, 0, payload, payload_off, dev_status, true),
                                  (const uint8_t *)workspace, s));
            marks.window(first, end, 2);
            KVC_TRY(launch_tensor(plan, 1, true, quant_batch(plan, reqs, first, end, lead, 1, payload, payload_off, dev_status, true),
                                  (const uint8_t *)workspace, s));
            marks.window(first, end, 3);
        } else {
            // launch by launch (K before V, widths ascending) over the requests of the window together
            CoderItem items[kCoderBatch][kTableSlots];
            const int waves = share ? shared_waves(plan, reqs, first, end) : 0;
            for (int k = 0; k < end - first; ++k) {
                const int i = window_item(first, end, lead, k);
                coder_items(plan, all, &reqs[i], (uint8_t *)payload + payload_off[i], (long long)(payload_off[i + 1] - payload_off[i]), i - first, waves,
                            items[k]);
            }
            CoderBatch none = coder_batch(plan, all, &reqs[lead], first, workspace, out_bytes, dev_status);
            none.waves = waves;
            // the first launch: K of the narrowest width, or K and V; it builds the tables of all
            CoderBatch b = none;
            for (int k = 0; k < end - first; ++k)
                for (int j = 0; j < (share ? 2 : 1); ++j) add_item(b, all.of[j], items[k][j]);
            b.builders = none.builders = all.n * kCandidates;          // (a launch has a table of its own)
            if (builders_apart(b, all.of[0], share ? 2 : 0, dt, none.builders)) b.apart = none.apart = none.builders;
            b.front = (unsigned)none.apart;
            marks.window(first, end, 1);
            KVC_TRY(launch_encode_section(share ? 2 : 0, all.of[0].bits, all.of[0].group, dt, b, s));
            if (share) {
                marks.window(first, end, 2);
                marks.window(first, end, 3);
                first = end;
                continue;
            }
            for (int is_v = 0; is_v < 2; ++is_v) {
                for (int j = 1; j < all.n; ++j) {
                    if (all.of[j].is_v != is_v) continue;
                    b = none;
                    for (int k = 0; k < end - first; ++k) add_item(b, all.of[j], items[k][j]);
                    KVC_TRY(launch_encode_section(is_v, all.of[j].bits, all.of[j].group, dt, b, s));
                }
                marks.window(first, end, 2 + is_v);
            }
        }
        first = end;
    }
    return KVC_OK;
}

extern "C" int kvc_compress(const kvc_plan_t *plan, const kvc_request *reqs, int32_t n, void *payload,
                            const uint64_t *payload_off, uint64_t *out_bytes, int32_t *dev_status,
                            void *workspace, void *hip_stream)
{
    return compress_on(plan, reqs, n, payload, payload_off, out_bytes, dev_status, workspace, (hipStream_t)hip_stream);
}

// ---- kvc_compress for callers that cannot allocate: the workspace is a static device array ----

// Every GPU the library runs on holds its own copy of this array until the process ends.  In host
// code the name is only a handle for hipGetSymbolAddress; the address it returns, one per device,
// is what the kernels and fills receive.
static __device__ __align__(256) unsigned char scratch[KVC_STATIC_WORKSPACE_BYTES];

static const int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_lock;

// the current device's copy of `scratch` (looked up once per device)
static int static_workspace(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return KVC_ERR_DEVICE;
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return KVC_ERR_DEVICE;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return KVC_OK;
}

extern "C" int kvc_compress_static(const kvc_plan_t *plan, const kvc_request *reqs, int32_t n, void *payload,
                                   const uint64_t *payload_off, uint64_t *out_bytes, int32_t *dev_status,
                                   void *hip_stream)
{
    if (!plan) return KVC_ERR_ARG;
    if (plan->blob_bytes) return KVC_ERR_UNSUPPORTED;      // width tables live in a caller workspace (kvc_workspace_init)
    if (kvc_workspace_size(plan) > (size_t)KVC_STATIC_WORKSPACE_BYTES) return KVC_ERR_CAPACITY;
    void *ws = nullptr;
    KVC_TRY(static_workspace(&ws));
    return compress_on(plan, reqs, n, payload, payload_off, out_bytes, dev_status, ws, (hipStream_t)hip_stream);
}

extern "C" int kvc_decompress(const kvc_plan_t *plan, const void *payload, const uint64_t *payload_off,
                              const kvc_request *dst, int32_t n, int32_t *dev_status, void *workspace,
                              void *hip_stream)
{
    KVC_TRY(check_batch(plan, dst, n, payload, payload_off, workspace));
    if (!dev_status || ((uintptr_t)dev_status & 3)) return KVC_ERR_ARG;
    const kvc_strategy &st = plan->strat;
    for (int i = 0; i < n; ++i) {
        Geometry g;
        geometry(plan, dst[i].tokens, &g);
        const long long cap = (long long)(payload_off[i + 1] - payload_off[i]);
        if (cap < kHeader || (!st.codec && cap < g.total) || (st.codec && cap < g.off_codes_k)) return KVC_ERR_CAPACITY;
        if (st.codec && !places_fit(g)) return KVC_ERR_UNSUPPORTED;
    }
    hipStream_t s = (hipStream_t)hip_stream;
    const int dt = plan->model.dtype;
    const Marks marks(plan, s);
    marks.at(0, 0);
    marks.window(0, n, 0);                     // (the checks of all requests come first)
    if (small_call(plan, dst, n)) {
        marks.window(0, n, 1);
        SmallDecompressArgs sd;
        memset(&sd, 0, sizeof sd);
        for (int i = 0; i < n; ++i) {
            Geometry g;
            geometry(plan, dst[i].tokens, &g);
            uint8_t *pl = (uint8_t *)const_cast<void *>(payload) + payload_off[i];
            for (int is_v = 0; is_v < 2; ++is_v) sd.item[sd.n++] = quant_args(plan, &dst[i], is_v, pl, g, dev_status + i, false);
            sd.check[i].payload = (const uint32_t *)pl;
            make_header(plan, dst[i].tokens, g, &sd.check[i].expect);
        }
        sd.requests = n;
        KVC_TRY(launch_decompress_call(st.bits_k, dt, sd, s));
        marks.window(0, n, 2);
        marks.window(0, n, 3);
        return KVC_OK;
    }
    if (st.codec) {
        DecodeSetupArgs da;
        memset(&da, 0, sizeof da);
        da.mask = 0x03fff3ffu;                 // words 10/11 (total) and 26..31 (code sizes) depend on the data
        da.slots = table_slots(plan);
        for (int is_v = 0; is_v < 2; ++is_v)
            for (int w = 0; w < 4; ++w) {
                if (plan->has_table[is_v] ? plan->width_count[is_v][w] > 0 : kWidths[w] == (is_v ? st.bits_v : st.bits_k))
                    da.slot_mask |= 1 << (da.slots == kTableSlots ? 4 * is_v + w : is_v);
            }
        for (int first = 0; first < n; first += kDecodeSetupBatch) {
            da.n = n - first < kDecodeSetupBatch ? n - first : kDecodeSetupBatch;
            for (int j = 0; j < da.n; ++j) {
                const int i = first + j;
                Geometry g;
                geometry(plan, dst[i].tokens, &g);
                const uint8_t *pl = (const uint8_t *)payload + payload_off[i];
                DecodeSetupItem &it = da.item[j];
                memset(&it, 0, sizeof it);
                it.payload = (const uint32_t *)pl;
                make_header(plan, dst[i].tokens, g, &it.expect);
                it.off_aux = g.off_aux;
                if (plan->blob_bytes) {        // the payload's width tables must be the plan's
                    it.tables = pl + g.off_widths;
                    it.plan_tables = (const uint8_t *)workspace;
                    it.table_bytes = g.widths;
                }
                it.lut = (uint16_t *)((uint8_t *)workspace + plan->blob_bytes + (size_t)i * plan->ws_request + lut_offset(plan));
                it.status = dev_status + i;
            }
            KVC_TRY(launch_decode_setup(da, s));
        }
    } else {
        for (int first = 0; first < n; first += kCheckBatch) {
            CheckArgs ca;
            memset(&ca, 0, sizeof ca);
            ca.n = n - first < kCheckBatch ? n - first : kCheckBatch;
            for (int j = 0; j < ca.n; ++j) {
                const int i = first + j;
                Geometry g;
                geometry(plan, dst[i].tokens, &g);
                const uint8_t *pl = (const uint8_t *)payload + payload_off[i];
                CheckItem &it = ca.item[j];
                it.payload = (const uint32_t *)pl;
                make_header(plan, dst[i].tokens, g, &it.expect);
                if (plan->blob_bytes) {        // the payload's width tables must be the plan's
                    it.tables = pl + g.off_widths;
                    it.plan_tables = (const uint8_t *)workspace;
                    it.table_bytes = g.widths;
                }
                it.status = dev_status + i;
            }
            KVC_TRY(launch_decompress_prologue(ca, s));
        }
    }
    const int shared_limit = shared_window(plan, dst, n);
    const int coder_limit = common_widths(plan) == 2 ? shared_limit : coder_window(plan, dst, n);
    const CoderLaunches all = coder_launches(plan, (const uint8_t *)workspace);
    for (int first = 0; first < n;) {
        int lead;
        const int end = request_window(plan, dst, n, first, st.codec ? coder_limit : kQuantBatch, &lead);
        if (!st.codec) {
            marks.window(first, end, 1);
            KVC_TRY(launch_tensor(plan, 0, false, quant_batch(plan, dst, first, end, lead, 0, const_cast<void *>(payload), payload_off, dev_status, false),
                                  (const uint8_t *)workspace, s));
            marks.window(first, end, 2);
            KVC_TRY(launch_tensor(plan, 1, false, quant_batch(plan, dst, first, end, lead, 1, const_cast<void *>(payload), payload_off, dev_status, false),
                                  (const uint8_t *)workspace, s));
            marks.window(first, end, 3);
        } else {
            CoderItem items[kCoderBatch][kTableSlots];
            for (int k = 0; k < end - first; ++k) {
                const int i = window_item(first, end, lead, k);
                coder_items(plan, all, &dst[i], (uint8_t *)const_cast<void *>(payload) + payload_off[i], (long long)(payload_off[i + 1] - payload_off[i]),
                            i - first, 0, items[k]);
            }
            const CoderBatch none = coder_batch(plan, all, &dst[lead], first, workspace, nullptr, dev_status);
            marks.window(first, end, 1);
            if (widths_share(plan, dst, first, end, lead, shared_limit)) {
                // width by width, K and V together
                for (int w = 0; w < 4; ++w) {
                    CoderBatch b = none;
                    int kinds = 0;                        // bit 0: K, bit 1: V
                    for (int k = 0; k < end - first; ++k)
                        for (int j = 0; j < all.n; ++j)
                            if (all.of[j].bits == kWidths[3 - w]) {
                                add_item(b, all.of[j], items[k][j]);
                                kinds |= 1 << all.of[j].is_v;
                            }
                    if (b.n > 0) KVC_TRY(launch_decode_section(kinds == 3 ? 2 : kinds - 1, kWidths[3 - w], dt, b, s));
                }
                marks.window(first, end, 2);
                marks.window(first, end, 3);
                first = end;
                continue;
            }
            for (int is_v = 0; is_v < 2; ++is_v) {
                for (int j = 0; j < all.n; ++j) {
                    if (all.of[j].is_v != is_v) continue;
                    CoderBatch b = none;
                    for (int k = 0; k < end - first; ++k) add_item(b, all.of[j], items[k][j]);
                    KVC_TRY(launch_decode_section(is_v, all.of[j].bits, dt, b, s));
                }
                marks.window(first, end, 2 + is_v);
            }
        }
        first = end;
    }
    return KVC_OK;
}
