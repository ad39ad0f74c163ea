// Host runtime of the Encode stage (T5-v1.1-style text encoder): tensor table, workspace
// layout and the launch sequence of one forward pass.  Every arithmetic step runs in the
// kernels of gemm.hip, attention.hip, elementwise.hip and encoder.hip.
#include "../../include/encoder.h"
#include "dit_internal.h"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <unordered_map>
#include <vector>

using namespace dit;

namespace {
struct ETensor {
  std::string name;
  int rows_in, cols_out, kind;   // 0 matrix (bf16 [out_pad][ld]), 2 gain, 3 table (fp32)
  size_t off; int ld, rows_pad;
};
struct ETap { void* dst; size_t cap; };
inline size_t rup(size_t x, size_t a) { return (x + a - 1) / a * a; }
constexpr size_t PARTIAL_BYTES = (size_t)256 * 128 * 128 * 4;    // split-K scratch of the GEMM
}  // namespace

struct enc_ctx {
  enc_config cfg;
  int device = 0;
  hipStream_t stream = nullptr;
  std::vector<ETensor> tensors;
  std::unordered_map<std::string, int> index;
  size_t weight_bytes = 0;
  unsigned char* weights = nullptr;
  unsigned char* ws = nullptr;
  size_t ws_bytes = 0;
  mutable std::string err;
  std::map<std::string, ETap> taps;
  std::vector<unsigned char> host_meta;        // kept alive until the upload has been consumed
  hipEvent_t meta_done = nullptr;
  bool launch_refused = false;     // a product of the running call was outside the GEMM's limits
};

namespace {

dit_status efail(const enc_ctx* c, dit_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap; va_start(ap, fmt); vsnprintf(buf, sizeof buf, fmt, ap); va_end(ap);
  if (c) c->err = buf;
  return st;
}
#define EHIP(c, call)                                                                              \
  do {                                                                                             \
    hipError_t e_ = (call);                                                                        \
    if (e_ != hipSuccess) return efail(c, DIT_EDEVICE, "%s: %s", #call, hipGetErrorString(e_));    \
  } while (0)

void add_tensor(enc_ctx* c, const std::string& name, int rows_in, int cols_out, int kind) {
  ETensor t;
  t.name = name; t.rows_in = rows_in; t.cols_out = cols_out; t.kind = kind;
  t.off = c->weight_bytes; t.ld = 0; t.rows_pad = 0;
  if (kind == 0) {
    t.ld = (int)rup(rows_in, 64); t.rows_pad = (int)rup(cols_out, 256);
    c->weight_bytes += rup((size_t)t.rows_pad * t.ld * 2, 256);
  } else {
    c->weight_bytes += rup((size_t)rows_in * cols_out * 4, 256);
  }
  c->index[name] = (int)c->tensors.size();
  c->tensors.push_back(t);
}
const ETensor* find(const enc_ctx* c, const std::string& n) {
  auto it = c->index.find(n);
  return it == c->index.end() ? nullptr : &c->tensors[it->second];
}
const bf16_t* Wm(const enc_ctx* c, const std::string& n) { return (const bf16_t*)(c->weights + find(c, n)->off); }
const float* Wv(const enc_ctx* c, const std::string& n) { return (const float*)(c->weights + find(c, n)->off); }
int Wld(const enc_ctx* c, const std::string& n) { return find(c, n)->ld; }

uint64_t fnv(const std::string& s) {
  uint64_t h = 0xCBF29CE484222325ull;
  for (unsigned char ch : s) { h ^= ch; h *= 0x100000001B3ull; }
  return h;
}
uint64_t mix(uint64_t x) {
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
uint16_t h_f2bf(float f) {
  uint32_t u; memcpy(&u, &f, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

struct Layout {
  size_t meta, x, h, q, k, vt, o, act, bias, partial, total;
  // offsets inside meta
  size_t o_cu, o_vt_off, o_vt_col, o_tiles;
  int M, cols_pad, L, n_tiles;
};

bool lens_ok(int n_seq, const int* lens) {
  if (n_seq <= 0 || n_seq > 4096 || !lens) return false;
  long long tot = 0;
  for (int s = 0; s < n_seq; ++s) {
    if (lens[s] < 1 || lens[s] > ENC_MAX_LEN) return false;
    tot += lens[s];
  }
  return tot <= (1 << 20);
}

// host image of the index data of one call + workspace layout
void plan(const enc_ctx* c, int n_seq, const int* lens, Layout& L, std::vector<unsigned char>* meta) {
  const enc_config& g = c->cfg;
  const size_t d = g.d_model, inner = (size_t)g.n_heads * g.head_dim, dff = g.d_ff;
  std::vector<int> cu(1, 0), vt_off, vt_col;     // vt_col: column of the transposed values for each token
  std::vector<AttnTile> tiles;
  int col = 0, longest = 0;
  for (int s = 0; s < n_seq; ++s) {
    vt_off.push_back(col);
    for (int t = 0; t < lens[s]; ++t) vt_col.push_back(col + t);
    col += (int)rup(lens[s], 64);
    for (int q0 = 0; q0 < lens[s]; q0 += 128) tiles.push_back(AttnTile{s, q0});
    longest = std::max(longest, lens[s]);
    cu.push_back(cu.back() + lens[s]);
  }
  std::stable_sort(tiles.begin(), tiles.end(), [&](const AttnTile& a, const AttnTile& b) { return lens[a.seg] > lens[b.seg]; });
  L.M = cu.back(); L.cols_pad = col; L.L = longest; L.n_tiles = (int)tiles.size();
  size_t mo = 0;
  auto put = [&](const void* p, size_t bytes) {
    const size_t at = rup(mo, 256);
    if (meta) { meta->resize(at + std::max<size_t>(bytes, 4)); if (bytes) memcpy(meta->data() + at, p, bytes); }
    mo = at + std::max<size_t>(bytes, 4);
    return at;
  };
  L.o_cu = put(cu.data(), cu.size() * 4);
  L.o_vt_off = put(vt_off.data(), vt_off.size() * 4);
  L.o_vt_col = put(vt_col.data(), vt_col.size() * 4);
  L.o_tiles = put(tiles.data(), tiles.size() * sizeof(AttnTile));
  const size_t meta_bytes = rup(mo, 256);
  if (meta) meta->resize(meta_bytes);
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t at = o; o += rup(bytes, 256); return at; };
  const size_t M = L.M;
  L.meta = take(meta_bytes);
  L.x = take(M * d * 4);
  L.h = take(M * d * 2);
  L.q = take(M * inner * 2); L.k = take(M * inner * 2);
  L.vt = take(inner * (size_t)col * 2);
  L.o = take(M * inner * 2);
  L.act = take(M * dff * 2);
  L.bias = take((size_t)g.n_heads * (2 * (size_t)longest - 1) * 4);
  L.partial = take(PARTIAL_BYTES);
  L.total = o;
}

GemmProblem prob(const bf16_t* A, int lda, const bf16_t* W, int ldw, int M, int N, int K, int kind, void* out, int ldc) {
  GemmProblem p;
  p.A = A; p.lda = lda; p.W = W; p.ldw = ldw; p.bias = nullptr; p.M = M; p.N = N; p.K = K;
  p.out_kind = kind; p.out = out; p.ldc = ldc; p.gate = nullptr; p.gate_stride = 0; p.row_req = nullptr;
  p.tiles_m = p.tiles_n = p.tile_start = 0;
  p.qk = QkNorm{};
  return p;
}
void gemm(enc_ctx* c, float* partial, std::initializer_list<GemmProblem> ps, bool geglu = false) {
  GemmBatch b;
  b.n = 0; b.total_tiles = 0; b.geglu = geglu;
  for (const GemmProblem& p : ps) b.p[b.n++] = p;
  b.partial = partial; b.partial_bytes = PARTIAL_BYTES;
  if (launch_gemm(c->stream, b) < 0) c->launch_refused = true;     // reported by the call
}

dit_status tap(enc_ctx* c, const std::string& name, const void* src, size_t bytes) {
  auto it = c->taps.find(name);
  if (it == c->taps.end()) return DIT_OK;
  if (bytes > it->second.cap) return efail(c, DIT_ENOMEM, "tap %s needs %zu bytes, buffer has %zu", name.c_str(), bytes, it->second.cap);
  EHIP(c, hipMemcpyAsync(it->second.dst, src, bytes, hipMemcpyDeviceToDevice, c->stream));
  return DIT_OK;
}
#define ETAP(name, src, bytes)                                            \
  do {                                                                    \
    if (!c->taps.empty()) {                                               \
      dit_status st_ = tap(c, name, src, bytes);                          \
      if (st_ != DIT_OK) return st_;                                      \
    }                                                                     \
  } while (0)

}  // namespace

extern "C" {

dit_status enc_create(const enc_config* cfg, int device, void* hip_stream, enc_ctx** out) {
  if (!out) return DIT_EINVAL;
  *out = nullptr;
  if (!cfg) return DIT_EINVAL;
  const enc_config& g = *cfg;
  if (g.vocab <= 0 || g.n_layers <= 0 || g.n_heads <= 0) return DIT_EINVAL;
  if (g.d_model <= 0 || g.d_model % 256 || g.d_model > 8192 || g.d_ff <= 0 || g.d_ff % 256) return DIT_ESHAPE;
  if ((g.head_dim != 64 && g.head_dim != 128) || (g.n_heads * g.head_dim) % 256) return DIT_ESHAPE;
  enc_ctx* c = new enc_ctx();
  c->cfg = g; c->device = device; c->stream = (hipStream_t)hip_stream;
  const int d = g.d_model, inner = g.n_heads * g.head_dim, dff = g.d_ff;
  add_tensor(c, "embed", g.vocab, d, 3);
  add_tensor(c, "rel_bias", 32, g.n_heads, 3);
  for (int l = 0; l < g.n_layers; ++l) {
    const std::string p = "l" + std::to_string(l);
    add_tensor(c, p + ".ln1.g", 1, d, 2);
    add_tensor(c, p + ".q.w", d, inner, 0);
    add_tensor(c, p + ".k.w", d, inner, 0);
    add_tensor(c, p + ".v.w", d, inner, 0);
    add_tensor(c, p + ".o.w", inner, d, 0);
    add_tensor(c, p + ".ln2.g", 1, d, 2);
    add_tensor(c, p + ".wi0.w", d, dff, 0);
    add_tensor(c, p + ".wi1.w", d, dff, 0);
    add_tensor(c, p + ".wo.w", dff, d, 0);
  }
  add_tensor(c, "final.g", 1, d, 2);
  *out = c;
  return DIT_OK;
}

void enc_destroy(enc_ctx* c) {
  if (!c) return;
  if (c->meta_done) { (void)hipEventSynchronize(c->meta_done); (void)hipEventDestroy(c->meta_done); }
  delete c;
}

const char* enc_last_error(const enc_ctx* c) { return c ? c->err.c_str() : "null context"; }
size_t enc_weight_bytes(const enc_ctx* c) { return c ? c->weight_bytes : 0; }

size_t enc_workspace_bytes(const enc_ctx* c, int n_seq, const int* lens) {
  if (!c || !lens_ok(n_seq, lens)) return 0;
  Layout L;
  plan(c, n_seq, lens, L, nullptr);
  return L.total;
}

dit_status enc_bind(enc_ctx* c, void* w, size_t wb, void* ws, size_t wsb) {
  if (!c) return DIT_EINVAL;
  if (!w || !ws) return efail(c, DIT_EINVAL, "null buffer");
  if (((uintptr_t)w & 255) || ((uintptr_t)ws & 255)) return efail(c, DIT_EINVAL, "buffers must be 256-byte aligned");
  if (wb < c->weight_bytes) return efail(c, DIT_ENOMEM, "weight arena has %zu bytes, needs %zu", wb, c->weight_bytes);
  c->weights = (unsigned char*)w; c->ws = (unsigned char*)ws; c->ws_bytes = wsb;
  return DIT_OK;
}

dit_status enc_init_weights(enc_ctx* c, uint64_t seed, float std) {
  if (!c) return DIT_EINVAL;
  if (!c->weights) return efail(c, DIT_EINVAL, "enc_bind has not been called");
  if (!(std >= 0.f) || !std::isfinite(std)) return efail(c, DIT_EINVAL, "std must be finite and non-negative");
  EHIP(c, hipSetDevice(c->device));
  EHIP(c, hipMemsetAsync(c->weights, 0, c->weight_bytes, c->stream));
  for (const ETensor& t : c->tensors) {
    const uint64_t key = mix(seed ^ (fnv(t.name) * 0x9E3779B97F4A7C15ull));
    if (t.kind == 0) launch_init_matrix(c->stream, (bf16_t*)(c->weights + t.off), t.cols_out, t.rows_in, t.ld, key, std);
    else if (t.kind == 3) launch_init_table_f32(c->stream, (float*)(c->weights + t.off), (long long)t.rows_in * t.cols_out, key, std);
    else launch_fill_f32(c->stream, (float*)(c->weights + t.off), t.cols_out, 1.0f);
  }
  EHIP(c, hipGetLastError());
  return DIT_OK;
}

int enc_tensor_count(const enc_ctx* c) { return c ? (int)c->tensors.size() : 0; }

dit_status enc_tensor_info(const enc_ctx* c, int i, char* name, size_t len, int* rows_in, int* cols_out, int* kind) {
  if (!c || i < 0 || i >= (int)c->tensors.size()) return DIT_EINVAL;
  const ETensor& t = c->tensors[i];
  if (name && len) { strncpy(name, t.name.c_str(), len - 1); name[len - 1] = 0; }
  if (rows_in) *rows_in = t.rows_in;
  if (cols_out) *cols_out = t.cols_out;
  if (kind) *kind = t.kind;
  return DIT_OK;
}

dit_status enc_set_tensor(enc_ctx* c, const char* name, const float* src, size_t n) {
  if (!c || !name || !src) return DIT_EINVAL;
  if (!c->weights) return efail(c, DIT_EINVAL, "enc_bind has not been called");
  const ETensor* t = find(c, name);
  if (!t) return efail(c, DIT_ENOTFOUND, "no tensor named %s", name);
  if (n != (size_t)t->rows_in * t->cols_out) return efail(c, DIT_ESHAPE, "%s has %d x %d elements", name, t->rows_in, t->cols_out);
  EHIP(c, hipSetDevice(c->device));
  EHIP(c, hipStreamSynchronize(c->stream));
  if (t->kind == 0) {
    std::vector<uint16_t> buf((size_t)t->rows_pad * t->ld, 0);
    for (int i = 0; i < t->rows_in; ++i)
      for (int o = 0; o < t->cols_out; ++o) buf[(size_t)o * t->ld + i] = h_f2bf(src[(size_t)i * t->cols_out + o]);
    EHIP(c, hipMemcpy(c->weights + t->off, buf.data(), buf.size() * 2, hipMemcpyHostToDevice));
  } else {
    EHIP(c, hipMemcpy(c->weights + t->off, src, n * 4, hipMemcpyHostToDevice));
  }
  return DIT_OK;
}

dit_status enc_get_tensor(enc_ctx* c, const char* name, float* dst, size_t n) {
  if (!c || !name || !dst) return DIT_EINVAL;
  if (!c->weights) return efail(c, DIT_EINVAL, "enc_bind has not been called");
  const ETensor* t = find(c, name);
  if (!t) return efail(c, DIT_ENOTFOUND, "no tensor named %s", name);
  if (n != (size_t)t->rows_in * t->cols_out) return efail(c, DIT_ESHAPE, "%s has %d x %d elements", name, t->rows_in, t->cols_out);
  EHIP(c, hipSetDevice(c->device));
  EHIP(c, hipStreamSynchronize(c->stream));
  if (t->kind == 0) {
    std::vector<uint16_t> buf((size_t)t->cols_out * t->ld);
    EHIP(c, hipMemcpy(buf.data(), c->weights + t->off, buf.size() * 2, hipMemcpyDeviceToHost));
    for (int i = 0; i < t->rows_in; ++i)
      for (int o = 0; o < t->cols_out; ++o) {
        const uint32_t u = (uint32_t)buf[(size_t)o * t->ld + i] << 16;
        memcpy(&dst[(size_t)i * t->cols_out + o], &u, 4);
      }
  } else {
    EHIP(c, hipMemcpy(dst, c->weights + t->off, n * 4, hipMemcpyDeviceToHost));
  }
  return DIT_OK;
}

dit_status enc_set_tap(enc_ctx* c, const char* point, void* dst, size_t bytes) {
  if (!c || !point || !dst) return DIT_EINVAL;
  c->taps[point] = ETap{dst, bytes};
  return DIT_OK;
}
void enc_clear_taps(enc_ctx* c) { if (c) c->taps.clear(); }

dit_status enc_forward(enc_ctx* c, int n_seq, const int* lens, const int* tokens, void* out_bf16, float* out_f32) {
  if (!c) return DIT_EINVAL;
  if (!c->weights || !c->ws) return efail(c, DIT_EINVAL, "enc_bind has not been called");
  if (!tokens || (!out_bf16 && !out_f32)) return efail(c, DIT_EINVAL, "null tokens or no output buffer");
  if (!lens_ok(n_seq, lens)) return efail(c, DIT_ESHAPE, "1..4096 sequences of 1..%d tokens, at most 2^20 tokens", (int)ENC_MAX_LEN);
  const enc_config& g = c->cfg;
  EHIP(c, hipSetDevice(c->device));
  c->launch_refused = false;
  // the previous call's host image must have been consumed before it is rebuilt
  if (c->meta_done) EHIP(c, hipEventSynchronize(c->meta_done));
  else EHIP(c, hipEventCreateWithFlags(&c->meta_done, hipEventDisableTiming));
  Layout L;
  plan(c, n_seq, lens, L, &c->host_meta);
  if (L.total > c->ws_bytes) return efail(c, DIT_ENOMEM, "workspace has %zu bytes, this call needs %zu", c->ws_bytes, L.total);
  hipStream_t s = c->stream;
  unsigned char* ws = c->ws;
  EHIP(c, hipMemcpyAsync(ws + L.meta, c->host_meta.data(), c->host_meta.size(), hipMemcpyHostToDevice, s));
  EHIP(c, hipEventRecord(c->meta_done, s));

  const int M = L.M, d = g.d_model, H = g.n_heads, dh = g.head_dim, inner = H * dh, dff = g.d_ff;
  float* x = (float*)(ws + L.x);
  bf16_t* h = (bf16_t*)(ws + L.h);
  bf16_t* q = (bf16_t*)(ws + L.q); bf16_t* k = (bf16_t*)(ws + L.k);
  bf16_t* vt = (bf16_t*)(ws + L.vt); bf16_t* o = (bf16_t*)(ws + L.o);
  bf16_t* act = (bf16_t*)(ws + L.act);
  float* bias = (float*)(ws + L.bias);
  float* partial = (float*)(ws + L.partial);
  const int* cu = (const int*)(ws + L.meta + L.o_cu);
  const int* vt_off = (const int*)(ws + L.meta + L.o_vt_off);
  const int* vt_col = (const int*)(ws + L.meta + L.o_vt_col);
  const AttnTile* tiles = (const AttnTile*)(ws + L.meta + L.o_tiles);

  launch_embed_gather(s, tokens, Wv(c, "embed"), x, M, d, g.vocab);
  launch_rel_bias_table(s, Wv(c, "rel_bias"), bias, H, L.L);
  // (pad columns of the transposed values: no product writes them)
  launch_fill_u16(s, vt, (long long)inner * L.cols_pad, 0);
  for (int l = 0; l < g.n_layers; ++l) {
    const std::string p = "l" + std::to_string(l);
    launch_rmsnorm(s, x, Wv(c, p + ".ln1.g"), h, nullptr, M, d);
    ETAP(p + ".ln1", h, (size_t)M * d * 2);
    // the values go out transposed, head by head, as the attention reads them
    GemmProblem pv = prob(h, d, Wm(c, p + ".v.w"), Wld(c, p + ".v.w"), M, inner, d, OUT_VT, nullptr, 0);
    pv.qk.nq = pv.qk.nk = 0; pv.qk.vt = vt; pv.qk.ldvt = L.cols_pad; pv.qk.vt_col = vt_col;
    gemm(c, partial, {prob(h, d, Wm(c, p + ".q.w"), Wld(c, p + ".q.w"), M, inner, d, OUT_BF16, q, inner),
                      prob(h, d, Wm(c, p + ".k.w"), Wld(c, p + ".k.w"), M, inner, d, OUT_BF16, k, inner),
                      pv});
    AttnArgs at;
    at.q = q; at.ldq = inner; at.k = k; at.ldk = inner; at.vt = vt; at.ldvt = L.cols_pad; at.o = o; at.ldo = inner;
    at.n_heads = H; at.head_dim = dh; at.cu_q = cu; at.cu_k = cu; at.vt_off = vt_off;
    at.tiles = tiles; at.n_tiles = L.n_tiles; at.q_per_tile = 128; at.o_row_map = nullptr;
    at.scale_log2 = 1.4426950408889634f;      // scores are not divided by sqrt(head_dim) in this encoder
    at.mode = 3; at.bias = bias; at.bias_L = L.L;
    launch_attention(s, at);
    ETAP(p + ".attn", o, (size_t)M * inner * 2);
    gemm(c, partial, {prob(o, inner, Wm(c, p + ".o.w"), Wld(c, p + ".o.w"), M, d, inner, OUT_RESID_F32, x, d)});
    ETAP(p + ".x_attn", x, (size_t)M * d * 4);
    launch_rmsnorm(s, x, Wv(c, p + ".ln2.g"), h, nullptr, M, d);
    gemm(c, partial, {prob(h, d, Wm(c, p + ".wi0.w"), Wld(c, p + ".wi0.w"), M, dff, d, OUT_BF16, act, dff),
                      prob(h, d, Wm(c, p + ".wi1.w"), Wld(c, p + ".wi1.w"), M, dff, d, OUT_BF16, act, dff)}, true);
    ETAP(p + ".act", act, (size_t)M * dff * 2);
    gemm(c, partial, {prob(act, dff, Wm(c, p + ".wo.w"), Wld(c, p + ".wo.w"), M, d, dff, OUT_RESID_F32, x, d)});
    ETAP(p + ".x_out", x, (size_t)M * d * 4);
  }
  launch_rmsnorm(s, x, Wv(c, "final.g"), (bf16_t*)out_bf16, out_f32, M, d);
  if (c->launch_refused) return efail(c, DIT_ESHAPE, "a matrix product of this call is outside the GEMM kernels' limits");
  EHIP(c, hipGetLastError());
  return DIT_OK;
}

}  // extern "C"
