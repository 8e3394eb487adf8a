// Device memory management, tensor views and the contraction engine.
//
// contract() evaluates C[lc] += alpha * sum A[la] B[lb] by classifying the
// labels (batch: in A, B and C; M: A and C; N: B and C; K: A and B), viewing
// each operand as a strided [batch][M][K] / [batch][K][N] / [batch][M][N]
// matrix when its axes can be merged, and copying it into a packed
// temporary otherwise.  The product itself runs on the FP64-MFMA complex
// GEMM kernel.
#include <algorithm>
#include <cstring>

#include <cmath>

#include "internal.h"

// ------------------------------------------------------------ allocation
namespace {
std::mutex g_contexts_mutex;  // taken before any context's in_call, which is only tried under it
std::vector<cclr_ctx*> g_contexts;

// releases the idle work memory of the other contexts on c's device that no call is using
void release_others(cclr_ctx* c) {
  std::lock_guard<std::mutex> lk(g_contexts_mutex);
  for (cclr_ctx* x : g_contexts) {
    if (x == c || x->device != c->device || !x->in_call.try_lock()) continue;
    x->arena.release_idle();
    x->in_call.unlock();
  }
}
}  // namespace

void register_context(cclr_ctx* c) {
  std::lock_guard<std::mutex> lk(g_contexts_mutex);
  g_contexts.push_back(c);
}

void unregister_context(cclr_ctx* c) {
  std::lock_guard<std::mutex> lk(g_contexts_mutex);
  g_contexts.erase(std::remove(g_contexts.begin(), g_contexts.end(), c), g_contexts.end());
}

// Where the cap or the device leaves no room, the context's own idle work
// memory is released and then that of the device's other contexts, before the
// request is refused: what contexts keep between calls costs no caller memory.
void DevBuf::alloc(cclr_ctx* c, size_t nbytes) {
  if (p && nbytes == bytes && ctx == c) return;  // same size: keep the allocation
  release();
  if (nbytes == 0) return;
  auto over_cap = [&]() { return c->opt.device_mem_cap && c->allocated + nbytes > c->opt.device_mem_cap; };
  if (over_cap()) c->arena.release_idle();
  if (over_cap())
    throw CclrError(CCLR_ENOMEM, "device memory cap exceeded (" + std::to_string(c->allocated + nbytes) +
                                     " > " + std::to_string(c->opt.device_mem_cap) + " bytes)");
  auto take = [&]() {
    if (c->dbg_fail_allocs > 0) {
      --c->dbg_fail_allocs;
      return false;
    }
    if (hipMalloc(&p, nbytes) == hipSuccess) return true;
    p = nullptr;
    (void)hipGetLastError();
    return false;
  };
  bool got = take();
  if (!got) {
    c->arena.release_idle();
    got = take();
  }
  if (!got) {
    release_others(c);
    got = take();
  }
  if (!got) throw CclrError(CCLR_ENOMEM, "hipMalloc of " + std::to_string(nbytes) + " bytes failed");
  ctx = c;
  bytes = nbytes;
  c->allocated += nbytes;
}

void DevBuf::release() {
  if (p) {
    (void)hipFree(p);
    if (ctx) ctx->allocated -= bytes;
  }
  p = nullptr;
  bytes = 0;
}

Arena::~Arena() {
  for (auto* b : chunks) delete b;
}

void* Arena::get(size_t bytes) {
  bytes = (bytes + 255) & ~size_t(255);
  if (ext) {
    if (bytes > ext_bytes - ext_used)
      throw CclrError(CCLR_ENOMEM, "work space of " + std::to_string(ext_bytes) + " bytes exhausted (" +
                                       std::to_string(ext_used + bytes) + " bytes needed so far)");
    void* p = ext + ext_used;
    ext_used += bytes;
    ext_peak = std::max(ext_peak, ext_used);
    return p;
  }
  while (cur < chunks.size()) {
    if (used[cur] + bytes <= chunks[cur]->bytes) {
      void* p = (char*)chunks[cur]->p + used[cur];
      used[cur] += bytes;
      return p;
    }
    if (cur + 1 < chunks.size()) ++cur;
    else break;
  }
  if (!chunks.empty() && used[cur] == 0 && chunks[cur]->bytes == 0) {  // an entry whose memory was released
    chunks[cur]->alloc(ctx, std::max(bytes, chunk_bytes));
    used[cur] = bytes;
    return chunks[cur]->p;
  }
  DevBuf* b = new DevBuf();
  try {
    b->alloc(ctx, std::max(bytes, chunk_bytes));
  } catch (...) {
    delete b;
    throw;
  }
  chunks.push_back(b);
  used.push_back(bytes);
  cur = chunks.size() - 1;
  return b->p;
}

void* Arena::try_get(size_t bytes) {
  bytes = (bytes + 255) & ~size_t(255);
  if (ext) return bytes <= ext_bytes - ext_used ? get(bytes) : nullptr;
  bool room = false;
  for (size_t k = cur; k < chunks.size() && !room; ++k) room = used[k] + bytes <= chunks[k]->bytes;
  if (!room && ctx->opt.device_mem_cap) return nullptr;
  try {
    return get(bytes);
  } catch (const CclrError&) {
    return nullptr;
  }
}

Arena::Mark Arena::mark() const {
  if (ext) return {size_t(-1), ext_used};
  return {cur, chunks.empty() ? 0 : used[cur]};
}

void Arena::reset(Mark m) {
  if (hold > 0) return;
  if (ext) {
    if (m.chunk == size_t(-1)) ext_used = m.top;
    return;
  }
  if (m.chunk == size_t(-1)) return;  // a mark of the external region
  for (size_t k = m.chunk + 1; k < chunks.size(); ++k) used[k] = 0;
  if (!chunks.empty()) used[m.chunk] = m.top;
  cur = m.chunk;
}

size_t Arena::idle() const {
  size_t b = 0;
  for (size_t k = chunks.size(); k > cur + 1 && used[k - 1] == 0; --k) b += chunks[k - 1]->bytes;
  return b;
}

void Arena::trim(size_t keep) {
  size_t left = idle();
  if (left <= keep) return;
  (void)hipDeviceSynchronize();
  while (left > keep && chunks.size() > cur + 1 && used.back() == 0) {
    left -= chunks.back()->bytes;
    delete chunks.back();
    chunks.pop_back();
    used.pop_back();
  }
}

void Arena::release_idle() {
  bool any = false;
  for (size_t k = 0; k < chunks.size(); ++k) any = any || (used[k] == 0 && chunks[k]->bytes > 0);
  if (!any) return;
  (void)hipDeviceSynchronize();  // queued work may still use what has been handed back
  for (size_t k = 0; k < chunks.size(); ++k)
    if (used[k] == 0) chunks[k]->release();
}

// idle arena memory a context keeps of a build's (4 GiB: what the build of
// the intermediates and a solve take at o = 12, v = 90), none under a memory
// cap; any allocation that finds no room gets it back
size_t arena_keep(const cclr_ctx* c) { return c->opt.device_mem_cap ? 0 : size_t(4) << 30; }

// How many of n vectors, each needing bytes_per_vec of working memory, fit
// in the device memory that is free or idle in the arena.  Idle memory stays
// for them: released here and taken again, it cost each response function at
// o = 20, v = 200 in BF16X3 (12 vectors, 48 slots) 1 to 4 s beside 1.15 s of
// work, since the driver hands out what it has just got back only once that is
// cleared.  Chunks of other sizes are released by the allocation that finds no
// room (DevBuf::alloc), and here under a cap, which they would eat into.
int fit_vectors(cclr_ctx* c, double bytes_per_vec, int n) {
  if (n <= 1) return n;
  if (c->opt.device_mem_cap) c->arena.trim();
  size_t fr = 0, tot = 0;
  HIPCHK(hipMemGetInfo(&fr, &tot));
  double budget = 0.8 * ((double)fr + (double)c->arena.idle());
  if (c->opt.device_mem_cap) {
    const double left = c->opt.device_mem_cap > c->allocated ? (double)(c->opt.device_mem_cap - c->allocated) : 0.0;
    budget = std::min(budget, left);
  }
  int fit = (int)std::max(1.0, std::min((double)n, std::floor(budget / std::max(bytes_per_vec, 1.0))));
  if (c->dbg_rhs_group > 0) fit = std::min(fit, c->dbg_rhs_group);
  return fit;
}

// ------------------------------------------------------------------ views
Ten ten(cplx* p, std::initializer_list<i64> dims) {
  Ten t;
  t.p = p;
  t.nd = (int)dims.size();
  int d = 0;
  for (i64 x : dims) t.dim[d++] = x;
  i64 s = 1;
  for (d = t.nd - 1; d >= 0; --d) {
    t.st[d] = s;
    s *= t.dim[d];
  }
  return t;
}

Ten ten(const DevBuf& b, std::initializer_list<i64> dims) { return ten(b.c(), dims); }

Ten reorder(const Ten& t, const char* from, const char* to) {
  Ten r = t;
  const int n = t.nd;
  REQUIRE((int)strlen(from) == n && (int)strlen(to) == n, CCLR_EINVAL, "reorder: label count");
  for (int d = 0; d < n; ++d) {
    const char* q = strchr(from, to[d]);
    REQUIRE(q, CCLR_EINVAL, "reorder: unknown label");
    const int s = (int)(q - from);
    r.dim[d] = t.dim[s];
    r.st[d] = t.st[s];
  }
  return r;
}

Ten scaled(const Ten& t, double re, double im) {
  Ten r = t;
  const double nr = t.sr * re - t.si * im, ni = t.sr * im + t.si * re;
  r.sr = nr;
  r.si = ni;
  return r;
}

Ten conjugated(const Ten& t) {
  // conj(s * conj?(x)) = conj(s) * conj(conj?(x))
  Ten r = t;
  r.conj = !t.conj;
  r.si = -t.si;
  return r;
}

Ten tmp(cclr_ctx* c, std::initializer_list<i64> dims) {
  i64 n = 1;
  for (i64 x : dims) n *= x;
  cplx* p = (cplx*)c->arena.get(sizeof(cplx) * (size_t)std::max<i64>(n, 1));
  return ten(p, dims);
}

void tzero(cclr_ctx* c, const Ten& t) {
  // only contiguous tensors are zeroed in one sweep
  i64 n = t.size();
  bool contig = true;
  i64 s = 1;
  for (int d = t.nd - 1; d >= 0; --d) {
    if (t.dim[d] != 1 && t.st[d] != s) contig = false;
    s *= t.dim[d];
  }
  if (contig) {
    launch_fill(t.p, n, cx(0.0), c->stream);
    return;
  }
  CopyArgs a{};
  a.nd = t.nd;
  for (int d = 0; d < t.nd; ++d) {
    a.dim[d] = t.dim[d];
    a.sd[d] = t.st[d];
    a.ss[d] = 0;
  }
  // alpha = 0 writes zeros without reading the source
  a.dst = t.p;
  a.src = t.p;
  a.ar = 0.0;
  a.ai = 0.0;
  a.conj = 0;
  a.acc = 0;
  a.total = n;
  launch_tcopy(a, c->stream);
}

// -------------------------------------------------------- copy / permute
static int lpos(const char* l, char ch) {
  const char* q = strchr(l, ch);
  return q ? (int)(q - l) : -1;
}

void tcopy(cclr_ctx* c, const Ten& dst, const char* ld, const Ten& src, const char* ls, cplx alpha,
           bool accumulate) {
  const int n = dst.nd;
  REQUIRE((int)strlen(ld) == n && (int)strlen(ls) == src.nd && src.nd == n, CCLR_EINVAL, "tcopy: labels");
  REQUIRE(!dst.conj && dst.sr == 1.0 && dst.si == 0.0, CCLR_EINVAL, "tcopy: scaled destination");
  CopyArgs a{};
  a.nd = n;
  i64 total = 1;
  for (int d = 0; d < n; ++d) {
    const int s = lpos(ls, ld[d]);
    REQUIRE(s >= 0 && src.dim[s] == dst.dim[d], CCLR_EINVAL, std::string("tcopy: label/dim mismatch ") + ld + " <- " + ls);
    a.dim[d] = dst.dim[d];
    a.sd[d] = dst.st[d];
    a.ss[d] = src.st[s];
    total *= dst.dim[d];
  }
  // alpha * s * op(x)
  a.ar = alpha.x * src.sr - alpha.y * src.si;
  a.ai = alpha.x * src.si + alpha.y * src.sr;
  a.conj = src.conj ? 1 : 0;
  a.acc = accumulate ? 1 : 0;
  a.dst = dst.p;
  a.src = src.p;
  a.total = total;
  launch_tcopy(a, c->stream);
}

// ---------------------------------------------------------------- engine
namespace {
struct Group {
  std::string labels;
  i64 size = 1;
  i64 stride = 0;
  bool ok = true;
};

// View the axes `g` (in this order) of tensor t with labels l as one merged
// axis.  Succeeds if consecutive axes are nested with matching strides.
Group merge(const Ten& t, const char* l, const std::string& g) {
  Group r;
  r.labels = g;
  if (g.empty()) return r;
  i64 size = 1;
  i64 expect = -1;
  for (int q = (int)g.size() - 1; q >= 0; --q) {
    const int d = lpos(l, g[q]);
    const i64 dim = t.dim[d], st = t.st[d];
    if (dim == 1) continue;
    if (expect < 0) {
      r.stride = st;
    } else if (st != expect) {
      r.ok = false;
    }
    expect = st * dim;
    size *= dim;
  }
  r.size = size;
  if (expect < 0) r.stride = 0;
  return r;
}

i64 labsize(const Ten& t, const char* l, char ch) { return t.dim[lpos(l, ch)]; }

// One label of a group: its extent and its strides in the operand (a) and in
// the output (c).
struct Lab {
  i64 dim, a, c;
};
struct Span {
  i64 size = 1, stride = 0;
  bool ok = true;
  bool unit() const { return size == 1 || stride == 1; }
};
// the labels of `mask` merged into one index (as merge() does), by operand (what 0) or output strides
Span span(const Lab* l, int n, unsigned mask, int what) {
  Span r;
  i64 expect = -1;
  for (int q = n - 1; q >= 0; --q) {
    if (!((mask >> q) & 1) || l[q].dim == 1) continue;
    const i64 st = what ? l[q].c : l[q].a;
    if (expect < 0) r.stride = st;
    else if (st != expect) r.ok = false;
    expect = st * l[q].dim;
    r.size *= l[q].dim;
  }
  return r;
}

// Chooses how contract() lowers a product whose tensors do not nest: 0 for
// one product with copies of the tensors that do not, else bit 0 / 1: copy A /
// B, bits 2-7 the M labels and bits 8-13 the N labels that become batch
// indices.  Estimated time in us: 3.5 for the product plus its padded work (16
// x 16 blocks at 45 TFLOP/s) or its bytes at 4 TB/s, a tensor without a unit
// stride in rows, columns or k counted four times (a 64-byte sector per
// element); 4 plus its bytes for each copy.  At o=10, v=80, four vectors, the
// copies of the doubles-sized outputs and of the W^ab_ej operand took 130 us of
// a 1150 us transform.
int cheapest_plan(const Ten& A, const char* la, const Ten& B, const char* lb, const Ten& C, const char* lc,
                  const std::string& Lm, const std::string& Ln, const std::string& Lk, bool okA0, bool okB0, bool okC0,
                  bool accumulate) {
  const int nm = (int)Lm.size(), nn = (int)Ln.size(), nk = (int)Lk.size();
  Lab M[6], N[6], KA[6], KB[6];
  for (int q = 0; q < nm; ++q) {
    const int d = lpos(la, Lm[q]);
    M[q] = {A.dim[d], A.st[d], C.st[lpos(lc, Lm[q])]};
  }
  for (int q = 0; q < nn; ++q) {
    const int d = lpos(lb, Ln[q]);
    N[q] = {B.dim[d], B.st[d], C.st[lpos(lc, Ln[q])]};
  }
  for (int q = 0; q < nk; ++q) {
    const int d = lpos(la, Lk[q]), e = lpos(lb, Lk[q]);
    KA[q] = {A.dim[d], A.st[d], 0};
    KB[q] = {B.dim[e], B.st[e], 0};
  }
  const unsigned am = (1u << nm) - 1, an = (1u << nn) - 1, ak = (1u << nk) - 1;
  const Span ka = span(KA, nk, ak, 0), kb = span(KB, nk, ak, 0);
  const double nA = (double)A.size(), nB = (double)B.size(), nC = (double)C.size(), k = (double)ka.size;
  const double us = 16.0 / 4e6;  // of one element at 4 TB/s
  auto up16 = [](i64 x) { return (double)((x + 15) / 16 * 16); };
  auto product = [&](i64 m, i64 n, double nb, double bytes) {
    return 3.5 + std::max(nb * up16(m) * up16(n) * k * 8.0 / 45e6, bytes * us);
  };
  const double cw = accumulate ? 2.0 : 1.0;  // reads and writes of an output element
  double best;
  {
    const Span m = span(M, nm, am, 0), n = span(N, nn, an, 0), mc = span(M, nm, am, 1), nc = span(N, nn, an, 1);
    const double fa = !okA0 || m.unit() || ka.unit() ? 1.0 : 4.0, fb = !okB0 || n.unit() || kb.unit() ? 1.0 : 4.0;
    const double fc = !okC0 ? 1.0 : cw * (mc.unit() || nc.unit() ? 1.0 : 4.0);
    best = product(m.size, n.size, 1.0, nA * fa + nB * fb + nC * fc);
    if (!okA0) best += 4.0 + 2.0 * nA * us;
    if (!okB0) best += 4.0 + 2.0 * nB * us;
    if (!okC0) best += 4.0 + (1.0 + cw) * nC * us;
  }
  int pick = 0;
  for (unsigned mm = 0; mm <= am; ++mm) {
    const Span mc = span(M, nm, am & ~mm, 1), bc = span(M, nm, mm, 1), ma = span(M, nm, am & ~mm, 0),
               ba = span(M, nm, mm, 0);
    if (!mc.ok || !bc.ok) continue;
    for (unsigned mn = 0; mn <= an; ++mn) {
      const Span nc = span(N, nn, an & ~mn, 1), dc = span(N, nn, mn, 1), nb = span(N, nn, an & ~mn, 0),
                 db = span(N, nn, mn, 0);
      if (!nc.ok || !dc.ok || bc.size * dc.size >= 65536) continue;
      for (int cp = 0; cp < 4; ++cp) {
        const bool ca = cp & 1, cb = cp & 2;
        if (!ca && !(ka.ok && ma.ok && ba.ok)) continue;
        if (!cb && !(kb.ok && nb.ok && db.ok)) continue;
        if (!mm && !mn && !cp) continue;
        const double fa = ca || ma.unit() || ka.unit() ? 1.0 : 4.0, fb = cb || nb.unit() || kb.unit() ? 1.0 : 4.0;
        const double fc = cw * (mc.unit() || nc.unit() ? 1.0 : 4.0);
        double t = product(mc.size, nc.size, (double)(bc.size * dc.size), nA * fa + nB * fb + nC * fc);
        if (ca) t += 4.0 + 2.0 * nA * us;
        if (cb) t += 4.0 + 2.0 * nB * us;
        if (t < best) {
          best = t;
          pick = cp | (int)(mm << 2) | (int)(mn << 8);
        }
      }
    }
  }
  return pick;
}
}  // namespace

void contract(cclr_ctx* c, cplx alpha, const Ten& A, const char* la, const Ten& B, const char* lb, const Ten& C,
              const char* lc, bool accumulate) {
  REQUIRE((int)strlen(la) == A.nd && (int)strlen(lb) == B.nd && (int)strlen(lc) == C.nd, CCLR_EINVAL,
          std::string("contract: label count ") + la + "," + lb + "->" + lc);
  REQUIRE(!C.conj && C.sr == 1.0 && C.si == 0.0, CCLR_EINVAL, "contract: scaled output");
  std::string Lb, Lm, Ln, Lk;
  for (const char* p = lc; *p; ++p) {
    const bool inA = lpos(la, *p) >= 0, inB = lpos(lb, *p) >= 0;
    REQUIRE(inA || inB, CCLR_EINVAL, std::string("contract: output label not in inputs: ") + lc);
    if (inA && inB) Lb += *p;
    else if (inA) Lm += *p;
    else Ln += *p;
  }
  for (const char* p = la; *p; ++p) {
    if (lpos(lc, *p) < 0) {
      REQUIRE(lpos(lb, *p) >= 0, CCLR_EINVAL, std::string("contract: unsummed label ") + la);
      Lk += *p;
    }
  }
  for (const char* p = lb; *p; ++p)
    if (lpos(lc, *p) < 0) REQUIRE(lpos(la, *p) >= 0, CCLR_EINVAL, std::string("contract: unsummed label ") + lb);
  // sizes must agree
  auto chk = [&](const std::string& g) {
    for (char ch : g) {
      i64 s = -1;
      if (lpos(la, ch) >= 0) s = labsize(A, la, ch);
      if (lpos(lb, ch) >= 0) REQUIRE(s < 0 || labsize(B, lb, ch) == s, CCLR_EINVAL, "contract: size mismatch");
      if (lpos(lc, ch) >= 0 && s >= 0) REQUIRE(labsize(C, lc, ch) == s, CCLR_EINVAL, "contract: size mismatch");
    }
  };
  chk(Lb), chk(Lm), chk(Ln), chk(Lk);

  // Without shared batch labels, output labels of one operand that break the
  // nesting of the M (or N) group can become a batch index of their own (the
  // other operand gets stride 0), which avoids copying operands or the output;
  // an operand may also be copied into the order the plan wants.  Where the
  // tensors as they are do not give one product, the plan of least estimated
  // time is taken.
  if (Lb.empty()) {
    struct Plan {
      std::string sm, rm, sn, rn;
      bool ca = false, cb = false;
    } best;
    const bool okA0 = merge(A, la, Lk).ok && merge(A, la, Lm).ok, okB0 = merge(B, lb, Lk).ok && merge(B, lb, Ln).ok,
               okC0 = merge(C, lc, Lm).ok && merge(C, lc, Ln).ok;
    const int pick = okA0 && okB0 && okC0 ? 0 : cheapest_plan(A, la, B, lb, C, lc, Lm, Ln, Lk, okA0, okB0, okC0, accumulate);
    if (pick) {
      const unsigned mm = (pick >> 2) & 63, mn = (pick >> 8) & 63;
      for (int q = 0; q < (int)Lm.size(); ++q) ((mm >> q) & 1 ? best.sm : best.rm) += Lm[q];
      for (int q = 0; q < (int)Ln.size(); ++q) ((mn >> q) & 1 ? best.sn : best.rn) += Ln[q];
      best.ca = pick & 1;
      best.cb = pick & 2;
      Arena::Mark mk = c->arena.mark();
      Ten Aw = A, Bw = B;
      std::string law = la, lbw = lb;
      auto relayout = [&](const Ten& X, const char* lx, const std::string& order, Ten& out, std::string& lout) {
        i64 n = 1;
        for (char ch : order) n *= labsize(X, lx, ch);
        Ten T;
        T.p = (cplx*)c->arena.get(sizeof(cplx) * (size_t)std::max<i64>(n, 1));
        T.nd = (int)order.size();
        i64 st = 1;
        for (int d = T.nd - 1; d >= 0; --d) {
          T.dim[d] = labsize(X, lx, order[d]);
          T.st[d] = st;
          st *= T.dim[d];
        }
        tcopy(c, T, order.c_str(), X, lx, cx(1.0), false);
        out = T;
        lout = order;
      };
      if (best.ca) relayout(A, la, best.sm + best.rm + Lk, Aw, law);
      if (best.cb) relayout(B, lb, best.sn + Lk + best.rn, Bw, lbw);
      const Group Am2 = merge(Aw, law.c_str(), best.rm), Ak2 = merge(Aw, law.c_str(), Lk),
                  As = merge(Aw, law.c_str(), best.sm);
      const Group Bn2 = merge(Bw, lbw.c_str(), best.rn), Bk2 = merge(Bw, lbw.c_str(), Lk),
                  Bs = merge(Bw, lbw.c_str(), best.sn);
      const Group Cm2 = merge(C, lc, best.rm), Cn2 = merge(C, lc, best.rn), Cs1 = merge(C, lc, best.sn),
                  Cs2 = merge(C, lc, best.sm);
      // a copied operand already carries its scale and conjugation
      const double sr = Aw.sr * Bw.sr - Aw.si * Bw.si, si = Aw.sr * Bw.si + Aw.si * Bw.sr;
      GemmArgs g{};
      g.M = (int)Am2.size;
      g.N = (int)Bn2.size;
      g.K = (int)Ak2.size;
      g.nb2 = (int)Cs2.size;
      g.batch = (int)(Cs1.size * Cs2.size);
      g.A = Aw.p; g.sAb = 0; g.sAb2 = As.stride; g.sAm = Am2.stride; g.sAk = Ak2.stride; g.conjA = Aw.conj;
      g.B = Bw.p; g.sBb = Bs.stride; g.sBb2 = 0; g.sBk = Bk2.stride; g.sBn = Bn2.stride; g.conjB = Bw.conj;
      g.C = C.p; g.sCb = Cs1.stride; g.sCb2 = Cs2.stride; g.sCm = Cm2.stride; g.sCn = Cn2.stride;
      g.ar = alpha.x * sr - alpha.y * si;
      g.ai = alpha.x * si + alpha.y * sr;
      g.beta = accumulate ? 1 : 0;
      REQUIRE(Am2.size < (1ll << 31) && Bn2.size < (1ll << 31) && Ak2.size < (1ll << 31), CCLR_EINVAL,
              "contract: dimension too large for one GEMM");
      if (g.K == 0) {
        if (!accumulate) tzero(c, C);
      } else {
        run_gemm(c, g);
      }
      c->arena.reset(mk);
      return;
    }
  }
  Arena::Mark mk = c->arena.mark();
  // ---- A as [b][m][k]
  Group Ab = merge(A, la, Lb), Am = merge(A, la, Lm), Ak = merge(A, la, Lk);
  Ten Aw = A;
  std::string law = la;
  if (!(Ab.ok && Am.ok && Ak.ok)) {
    std::string nl = Lb + Lm + Lk;
    Ten T = tmp(c, {1});
    // allocate contiguous buffer
    i64 n = 1;
    for (char ch : nl) n *= labsize(A, la, ch);
    T.p = (cplx*)c->arena.get(sizeof(cplx) * (size_t)n);
    T.nd = (int)nl.size();
    i64 s = 1;
    for (int d = T.nd - 1; d >= 0; --d) {
      T.dim[d] = labsize(A, la, nl[d]);
      T.st[d] = s;
      s *= T.dim[d];
    }
    tcopy(c, T, nl.c_str(), A, la, cx(1.0), false);
    Aw = T;
    law = nl;
    Ab = merge(Aw, law.c_str(), Lb), Am = merge(Aw, law.c_str(), Lm), Ak = merge(Aw, law.c_str(), Lk);
  }
  // ---- B as [b][k][n]
  Group Bb = merge(B, lb, Lb), Bk = merge(B, lb, Lk), Bn = merge(B, lb, Ln);
  Ten Bw = B;
  std::string lbw = lb;
  if (!(Bb.ok && Bk.ok && Bn.ok)) {
    std::string nl = Lb + Lk + Ln;
    i64 n = 1;
    for (char ch : nl) n *= labsize(B, lb, ch);
    Ten T;
    T.p = (cplx*)c->arena.get(sizeof(cplx) * (size_t)n);
    T.nd = (int)nl.size();
    i64 s = 1;
    for (int d = T.nd - 1; d >= 0; --d) {
      T.dim[d] = labsize(B, lb, nl[d]);
      T.st[d] = s;
      s *= T.dim[d];
    }
    tcopy(c, T, nl.c_str(), B, lb, cx(1.0), false);
    Bw = T;
    lbw = nl;
    Bb = merge(Bw, lbw.c_str(), Lb), Bk = merge(Bw, lbw.c_str(), Lk), Bn = merge(Bw, lbw.c_str(), Ln);
  }
  // ---- C as [b][m][n]
  Group Cb = merge(C, lc, Lb), Cm = merge(C, lc, Lm), Cn = merge(C, lc, Ln);
  // a copied operand already carries its scale and conjugation
  const double sr = Aw.sr * Bw.sr - Aw.si * Bw.si, si = Aw.sr * Bw.si + Aw.si * Bw.sr;
  const cplx al = cx(alpha.x * sr - alpha.y * si, alpha.x * si + alpha.y * sr);

  GemmArgs g{};
  g.M = (int)Am.size;
  g.N = (int)Bn.size;
  g.K = (int)Ak.size;
  g.batch = (int)Ab.size;
  g.A = Aw.p; g.sAb = Ab.stride; g.sAm = Am.stride; g.sAk = Ak.stride; g.conjA = Aw.conj;
  g.B = Bw.p; g.sBb = Bb.stride; g.sBk = Bk.stride; g.sBn = Bn.stride; g.conjB = Bw.conj;
  REQUIRE(Am.size < (1ll << 31) && Bn.size < (1ll << 31) && Ak.size < (1ll << 31) && Ab.size < 65536, CCLR_EINVAL,
          "contract: dimension too large for one GEMM");

  if (Cb.ok && Cm.ok && Cn.ok) {
    g.C = C.p; g.sCb = Cb.stride; g.sCm = Cm.stride; g.sCn = Cn.stride;
    g.ar = al.x; g.ai = al.y; g.beta = accumulate ? 1 : 0;
    if (g.K == 0) {
      if (!accumulate) tzero(c, C);
    } else {
      run_gemm(c, g);
    }
  } else {
    std::string nl = Lb + Lm + Ln;
    i64 n = 1;
    for (char ch : nl) n *= labsize(C, lc, ch);
    Ten T;
    T.p = (cplx*)c->arena.get(sizeof(cplx) * (size_t)n);
    T.nd = (int)nl.size();
    i64 s = 1;
    for (int d = T.nd - 1; d >= 0; --d) {
      T.dim[d] = labsize(C, lc, nl[d]);
      T.st[d] = s;
      s *= T.dim[d];
    }
    g.C = T.p;
    g.sCb = g.M * (i64)g.N;
    g.sCm = g.N;
    g.sCn = 1;
    g.ar = al.x; g.ai = al.y; g.beta = 0;
    run_gemm(c, g);
    tcopy(c, C, lc, T, nl.c_str(), cx(1.0), accumulate);
  }
  c->arena.reset(mk);
}

// g with its B side split already: splits the A side and multiplies.  What is
// left of the arena goes to the split first: the product can do without cut
// tiles and their partial sums.
void split_product(cclr_ctx* c, const GemmArgs& g, int form, const SplitMat& B) {
  Arena::Mark mk = c->arena.mark();
  const SplitPlan whole = split_plan(g.M, g.N, g.K, form, false);
  const size_t need = split_bytes(g.M, g.K, form, 0, whole.bm);
  SplitPlan p = split_plan(g.M, g.N, g.K, form, true);
  const size_t want = split_bytes(g.M, g.K, form, 0, p.bm);
  void* wa = want > need ? c->arena.try_get(want) : nullptr;
  if (!wa) wa = c->arena.get(need), p = want > need ? whole : p;
  void* W = p.cutters > 0 ? c->arena.try_get(split_workspace(p)) : nullptr;
  if (!W) p = whole;
  const SplitMat A = launch_split(g.M, g.K, g.A, g.sAm, g.sAk, g.conjA, wa, form, 0, c->stream, p.bm);
  launch_split_gemm(A, B, g.C, g.sCm, g.sCn, g.ar, g.ai, g.beta, p, W, c->stream);
  c->arena.reset(mk);
}

// GEMM dispatch: products whose output covers too few 64x64 tiles to occupy
// the 256 compute units split the reduction into chunks that write partial
// products to a workspace, summed in a fixed order afterwards.
// form: the kernel that ran (FP64 variant >= 0, -1 short-reduction VALU
// kernel, -2 split-K with the default variant, -3 reduced precision, -4
// short-output VALU kernel, -5 reduced precision on pre-split FP32 planes, -6
// short-output VALU kernel on a long operand contiguous in k, -7 small
// products straight from registers, -8 even split over the compute units)
static void run_gemm_form(cclr_ctx* c, const GemmArgs& g, int& form);
void run_gemm(cclr_ctx* c, const GemmArgs& g) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0 || g.K <= 0) return;
  int form = 0;
  if (!c->gemm_trace) {
    run_gemm_form(c, g, form);
    return;
  }
  hipEvent_t e0, e1;
  HIPCHK(hipEventCreate(&e0));
  HIPCHK(hipEventCreate(&e1));
  HIPCHK(hipEventRecord(e0, c->stream));
  run_gemm_form(c, g, form);
  HIPCHK(hipEventRecord(e1, c->stream));
  HIPCHK(hipEventSynchronize(e1));
  float ms = 0.f;
  HIPCHK(hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  char line[384];
  snprintf(line, sizeof line,
           "%dx%dx%d b%d sA(%lld,%lld) sB(%lld,%lld) sC(%lld,%lld) sb(%lld,%lld,%lld) beta %d form %d %.4f ms "
           "%.2f TFLOP/s",
           g.M, g.N, g.K, g.batch, (long long)g.sAm, (long long)g.sAk, (long long)g.sBk, (long long)g.sBn,
           (long long)g.sCm, (long long)g.sCn, (long long)g.sAb, (long long)g.sBb, (long long)g.sCb, g.beta, form, ms,
           8.0 * g.M * (double)g.N * g.K * g.batch / (ms * 1e-3) / 1e12);
  c->gemm_trace_log.push_back(line);
}

// C^T = B^T A^T: the same product with the roles of m and n exchanged
static GemmArgs transposed(const GemmArgs& g0) {
  GemmArgs g = g0;
  g.M = g0.N; g.N = g0.M;
  g.A = g0.B; g.sAb = g0.sBb; g.sAb2 = g0.sBb2; g.sAm = g0.sBn; g.sAk = g0.sBk; g.conjA = g0.conjB;
  g.B = g0.A; g.sBb = g0.sAb; g.sBb2 = g0.sAb2; g.sBk = g0.sAk; g.sBn = g0.sAm; g.conjB = g0.conjA;
  g.sCm = g0.sCn; g.sCn = g0.sCm;
  return g;
}

// dst[b][e][r][q] (+)= src[b][e][r][q] between two strided 4-index views
// (b, e: the two levels of a GEMM batch)
static void copy4(cclr_ctx* c, const i64 (&dim)[4], cplx* dst, const i64 (&sd)[4], const cplx* src,
                  const i64 (&ss)[4], bool acc) {
  CopyArgs a{};
  a.nd = 4;
  a.total = 1;
  for (int d = 0; d < 4; ++d) {
    a.dim[d] = dim[d];
    a.sd[d] = sd[d];
    a.ss[d] = ss[d];
    a.total *= dim[d];
  }
  a.dst = dst;
  a.src = src;
  a.ar = 1.0;
  a.ai = 0.0;
  a.conj = 0;
  a.acc = acc ? 1 : 0;
  launch_tcopy(a, c->stream);
}

constexpr int kFormFrag = -7, kFormEven = -8;

// Products for the register kernel (gemm_frag.hip), counted in 16 x 16 output
// blocks f and 16-deep K tiles kt.  Times in us, this kernel against the one
// that ran before:
//  * up to 5120 block tiles, where every other kernel waits on one chain of
//    loads per workgroup: 16x4x480 9 against 44 (64x32 tiles), 93x31x465 9
//    against 76 (128x32), 465x93x31 4 against 37 (vector ALU), 558x186x186 8
//    against 34 (64x64); at 7128 (45x3160x45, batch 4) 22 against 12;
//  * long reductions with at most 96 blocks, or at most 128 where one side is
//    at most 48, or up to 14000 block tiles: 10x40x31600 13 against 59,
//    130x10x83850 43 against 195, 80x80x3600, batch 3 29 against 43 (evenly
//    split), 144x144x8100 44 against 47, 96x96x1000, batch 6 23 against 27;
//    beyond, 90x90x5940, batch 4 (144 blocks) 59 against 52.  Up to 4 columns
//    the vector kernels stay: 80x4x800, batch 80, 27 against 31, but 800x4x800
//    13 against 9;
//  * shorter reductions with one side at most 16 (above K = 32 and 4 columns),
//    which reads the long operand once at the copy rate: 83850x10x10 11 against
//    31, 14400x16x16, batch 32, 39 against 52, 97200x12x90 32 against 48 (32
//    columns), 83850x10x130 41 against 65, 1728000x16x120 908 against 944.
// Outputs 17 to 32 wide with more than 128 blocks stay on the 32-column tiles.
static bool frag_may_pay(const GemmArgs& g) {
  if (g.kchunk > 0 || g.batch >= 65536) return false;
  const i64 f = (i64)((g.M + 15) / 16) * ((g.N + 15) / 16) * g.batch, kt = (g.K + 15) / 16;
  const int lo = std::min(g.M, g.N);
  if (g.K > 32 && lo > 16 && lo <= 32 && f > 128) return false;
  if (f * kt <= 5120) return true;
  if (g.K >= 512) return lo > 4 && ((lo <= 48 && f <= 128) || f <= 40 || (lo > 16 && (f <= 96 || f * kt <= 14000)));
  return lo <= 16 && (g.K <= 32 || lo > 4) && f < (i64(1) << 22);
}

static void small_product(cclr_ctx* c, const GemmArgs& g) {
  // lanes run along n: the unit-stride index of the output
  const GemmArgs h = (g.sCn != 1 && g.sCm == 1) ? transposed(g) : g;
  const FragPlan p = frag_plan(h);
  Arena::Mark mk = c->arena.mark();
  cplx* W = p.S > 1 ? (cplx*)c->arena.get(sizeof(cplx) * (size_t)h.batch * p.S * h.M * (size_t)h.N) : nullptr;
  launch_zgemm_frag(h, p, W, c->stream);
  c->arena.reset(mk);
}

// The short-reduction kernel runs 256 lanes along n: where they are mostly
// idle the MFMA tiles are faster (3600x320x10: 9 us on 64x32 tiles against
// 18; 120x120x16, batch 240: 21 on 64x64 tiles against 31), where they are
// full it is (90x8100x12, batch 12: 37 against 43 us).
static bool smallk_may_pay(const GemmArgs& g) {
  const i64 n = (g.sCn != 1 && g.sCm == 1) ? g.M : g.N;
  return 4 * n >= 3 * ((n + 255) / 256 * 256);
}

// Time of a product in us by the work it puts on the busiest compute unit;
// the constants are fitted to measurements at o = 10 .. 20 (a K tile of 16 on
// a 16 fm x 64 tile takes 0.478 fm us of a compute unit, 0.51 fm alone on it;
// one on a 128x128 direct-load tile 7.27 us; a partial sum is written and read
// at 4 TB/s).
static double even_cost(const SkPlan& p) {
  const double tau = (p.fm == 2 ? 0.495 : 0.478) * p.fm, alone = 0.51 * p.fm, round = 2.0 * p.nk * tau;
  const i64 full = p.whole / 512, rem = p.whole % 512;
  double t = (double)full * (round + 2.5);
  if (rem) t += 2.5 + (rem <= 256 ? p.nk * alone : round);
  if (p.cutters) {
    const double rest = (double)(p.tiles - p.whole), run = rest * p.nk / p.cutters;
    t += 2.5 + std::max(rest * p.nk * tau / 256.0, run * alone);
    t += 6.0 + (p.cutters + rest) * 2.0 * (16.0 * 64 * 16) * p.fm / 4e6;
  }
  return t;
}

// the same for whole rounds of 128x128 direct-load tiles
static double dma_cost(const GemmArgs& g) {
  const int K = g.kchunk > 0 ? g.kchunk : g.K;
  const i64 t = (i64)((g.M + 127) / 128) * ((g.N + 127) / 128) * g.batch;
  return (double)((t + 255) / 256) * (7.27 * ((K + 15) / 16) + 8.0);
}

// FP64 products of some length on the evenly split kernel, in the orientation
// and row count of least estimated time; false: not taken (short reductions,
// where the other tiles are as fast, or large products that fill whole rounds
// of 128x128 tiles)
static bool even_split(cclr_ctx* c, const GemmArgs& g0) {
  if (g0.K < (std::min(g0.M, g0.N) <= 32 ? 512 : 256) || g0.kchunk > 0) return false;
  const i64 most = (i64)((g0.M + 31) / 32) * ((g0.N + 31) / 32) * g0.batch;
  if (most >= (1ll << 30)) return false;
  const double dma = dma_cost(g0);
  // with two workgroups per compute unit, with one where the partial sums of
  // two have no room, and with whole tiles only
  for (int cutters : {512, 256, 0}) {
    double best = 1e300;
    SkPlan plan;
    bool trans = false;
    for (int o = 0; o < 2; ++o) {
      const GemmArgs g = o ? transposed(g0) : g0;
      for (int fm = 2; fm <= 6; ++fm) {
        const SkPlan p = sk_plan_for(g, fm, cutters);
        // stores along the unit-stride index where both orientations are as good
        const double t = even_cost(p) * (g.sCn == 1 ? 1.0 : 1.02);
        if (t < best) best = t, plan = p, trans = o;
      }
    }
    if (dma * 0.98 <= best) return false;
    // a few whole tiles leave most of the chip idle: the split-K kernels
    if (cutters == 0 && plan.tiles < 192) return false;
    Arena::Mark mk = c->arena.mark();
    cplx* W = nullptr;
    if (plan.cutters > 0 && !(W = (cplx*)c->arena.try_get(sk_workspace(plan)))) continue;
    launch_zgemm_sk(trans ? transposed(g0) : g0, plan, W, c->stream);
    c->arena.reset(mk);
    return true;
  }
  return false;
}

// two batch levels that are one: the first of extent 1, or each stride of it
// the second's times its extent
static bool one_level(const GemmArgs& g) {
  return g.nb2 > 1 && (g.batch == g.nb2 || (g.sAb == g.nb2 * g.sAb2 && g.sBb == g.nb2 * g.sBb2 && g.sCb == g.nb2 * g.sCb2));
}

static void run_gemm_form(cclr_ctx* c, const GemmArgs& g0, int& form) {
  form = -1;
  // the split along K takes one level: 200x200x38000 in a batch of 3 on the
  // second, in FP32, 3.9 ms without it and 0.6 with
  if (one_level(g0)) {
    GemmArgs h = g0;
    h.sAb = g0.sAb2, h.sBb = g0.sBb2, h.sCb = g0.sCb2;
    h.nb2 = 0;
    h.sAb2 = h.sBb2 = h.sCb2 = 0;
    run_gemm_form(c, h, form);
    return;
  }
  // An operand or output whose unit stride is a batch index would have every
  // tile (or every thread's row) touch one element per cache line of it:
  // such tensors are copied to a batch-outermost layout first, and the
  // output is added back afterwards.
  if (g0.kchunk == 0 && g0.batch >= 8) {
    const i64 M = g0.M, N = g0.N, K = g0.K;
    const i64 n2 = g0.nb2 > 1 ? g0.nb2 : 1, n1 = g0.batch / n2;
    auto inner = [&](i64 s1, i64 s2, i64 sz) { return sz > 1 && ((n1 > 1 && s1 == 1) || (n2 > 1 && s2 == 1)); };
    const bool ca = inner(g0.sAb, g0.sAb2, M * K), cb = inner(g0.sBb, g0.sBb2, K * N),
               cc = inner(g0.sCb, g0.sCb2, M * N);
    const i64 big = (i64)g0.batch * std::max({ca ? M * K : 0, cb ? K * N : 0, cc ? M * N : 0});
    if ((ca || cb || cc) && big >= (i64(1) << 20)) {
      Arena::Mark mk = c->arena.mark();
      GemmArgs h = g0;
      const i64 s2b = n2 > 1 ? 1 : 0;  // the second batch level's stride factor in the copies
      // a batch level that an input does not vary over (stride 0) is copied once
      auto outermost = [&](const cplx*& X, i64& s1, i64& s2, i64& sr, i64& sq, i64 r, i64 q) {
        const i64 d1 = s1 == 0 ? 1 : n1, d2 = s2b * s2 == 0 ? 1 : n2;
        cplx* t = (cplx*)c->arena.get(sizeof(cplx) * (size_t)(d1 * d2 * r * q));
        copy4(c, {d1, d2, r, q}, t, {d2 * r * q, r * q, q, 1}, X, {s1, s2b * s2, sr, sq}, false);
        X = t;
        s1 = s1 == 0 ? 0 : d2 * r * q;
        s2 = s2b * s2 == 0 ? 0 : r * q;
        sr = q;
        sq = 1;
      };
      if (ca) outermost(h.A, h.sAb, h.sAb2, h.sAm, h.sAk, M, K);
      if (cb) outermost(h.B, h.sBb, h.sBb2, h.sBk, h.sBn, K, N);
      if (cc) {
        cplx* t = (cplx*)c->arena.get(sizeof(cplx) * (size_t)(g0.batch * M * N));
        h.C = t; h.sCb = n2 * M * N; h.sCb2 = M * N; h.sCm = N; h.sCn = 1; h.beta = 0;
      }
      run_gemm_form(c, h, form);
      if (cc)
        copy4(c, {n1, n2, M, N}, g0.C, {g0.sCb, s2b * g0.sCb2, g0.sCm, g0.sCn}, h.C, {n2 * M * N, M * N, N, 1},
              g0.beta != 0);
      c->arena.reset(mk);
      return;
    }
  }
  // reduced-precision transforms take the small products in FP64 like the
  // others: those are bound by latency and memory, not by the arithmetic
  const bool frag = frag_may_pay(g0);
  if (g0.K <= 32) {
    if (frag) {
      form = kFormFrag;
      small_product(c, g0);
      return;
    }
    // (the MFMA tiles of a reduced-precision transform are FP32)
    if ((smallk_may_pay(g0) || c->sigma_prec != CCLR_FP64) && launch_zgemm_smallk(g0, c->stream)) return;
  }
  // the MFMA tiles are at least 32 columns but 64 (FP64) or 128 (FP32) rows
  // high: a product with a short m side (at most 32) and a long n side runs
  // transposed, so that its short side can take the 32-column tiles
  const GemmArgs g = (g0.M <= 32 && g0.N > 32) ? transposed(g0) : g0;
  {
    // at most 8 output columns, long operand contiguous in k: rows dotted along k
    int kc = 0, S = 0;
    if (rowdot_plan(g, kc, S)) {
      form = -6;
      Arena::Mark mk = c->arena.mark();
      cplx* W = S > 1 ? (cplx*)c->arena.get(sizeof(cplx) * (size_t)g.batch * S * g.M * (size_t)g.N) : nullptr;
      launch_zgemm_rowdot(g, kc, S, W, c->stream);
      c->arena.reset(mk);
      return;
    }
    if (frag) {
      form = kFormFrag;
      small_product(c, g0);
      return;
    }
    // at most 16 output columns: FP64 VALU rows instead of mostly empty MFMA tiles
    GemmArgs h;
    if (skinny_plan(g, h, kc, S)) {
      form = -4;
      Arena::Mark mk = c->arena.mark();
      cplx* W = S > 1 ? (cplx*)c->arena.get(sizeof(cplx) * (size_t)h.batch * S * h.M * (size_t)h.N) : nullptr;
      launch_zgemm_skinny(h, kc, S, W, c->stream);
      c->arena.reset(mk);
      return;
    }
  }
  // inside reduced-precision transforms the remaining products run on FP32 MFMA as well
  const bool lowp = c->sigma_prec != CCLR_FP64;
  if (!lowp && even_split(c, g)) {
    form = kFormEven;
    return;
  }
  const i64 tiles = (i64)((g.M + 63) / 64) * ((g.N + 63) / 64) * g.batch;
  if (g.nb2 <= 1 && tiles < 512 && g.K >= 512) {
    i64 S = std::min<i64>((1024 + tiles - 1) / tiles, g.K / 256);
    S = std::max<i64>(S, 2);
    i64 kc = (g.K + S - 1) / S;
    kc = (kc + 15) / 16 * 16;
    S = (g.K + kc - 1) / kc;
    if ((i64)g.batch * S < 65536) {
      Arena::Mark mk = c->arena.mark();
      cplx* W = (cplx*)c->arena.get(sizeof(cplx) * (size_t)(g.batch * S * g.M * (i64)g.N));
      GemmArgs h = g;
      h.kchunk = (int)kc;
      h.batch = (int)(g.batch * S);
      h.nb2 = 0;
      h.C = W;
      h.sCb = (i64)g.M * g.N;
      h.sCm = g.N;
      h.sCn = 1;
      h.ar = 1.0;
      h.ai = 0.0;
      h.beta = 0;
      form = lowp ? -3 : -2;
      if (lowp) launch_zgemm_lowp(h, CCLR_FP32, c->stream);
      else gemm_by_rule(c, h);
      launch_chunk_reduce(g, (int)S, W, c->stream);
      c->arena.reset(mk);
      return;
    }
  }
  if (lowp) {
    form = -3;
    // large single products: each operand converted once to the three FP32
    // Gauss planes, then the direct-load split kernel (the conversion passes
    // cost less than the gain over converting inside the K loop once both
    // output sides are a few hundred long)
    if (g.batch == 1 && g.kchunk == 0 && g.nb2 <= 1 && g.M >= 512 && g.N >= 512 && g.K >= 256) {
      form = -5;
      Arena::Mark mk = c->arena.mark();
      void* wb = c->arena.get(split_bytes(g.N, g.K, F32_G3, 1));
      const SplitMat B = launch_split(g.N, g.K, g.B, g.sBn, g.sBk, g.conjB, wb, F32_G3, 1, c->stream);
      split_product(c, g, F32_G3, B);
      c->arena.reset(mk);
      return;
    }
    launch_zgemm_lowp(g, CCLR_FP32, c->stream);
  } else {
    form = gemm_by_rule(c, g);
  }
}

void launch_gemm_choice(const GemmArgs& g, int choice, hipStream_t s) {
  if (choice >= kTransposedChoice) launch_zgemm_variant(transposed(g), choice - kTransposedChoice, s);
  else launch_zgemm_variant(g, choice, s);
}

// Tile of the products that neither the register nor the evenly split kernel
// takes: the least estimated time in us, 256 compute units taking one round of
// tiles after another.  The constants are fitted to one MI355X; nk K tiles of
// 16, t workgroups per 256:
//   64x64, one LDS buffer  t (1.98 nk + 1)   7140x7140x120 825 (measured 821)
//   128x32, one LDS buffer t (2.1 nk + 1)    2197000x10x130 1353 (1355)
//   64x32                  t (1.08 nk + 1)   130x130x130, batch 400 257 (255)
//   128x128 direct loads   t (7.27 nk + 8)   4000x4000x400 759 (756)
// Over 43 shapes (N from 10 to 40000, K from 28 to 4000, batches to 700) the
// choice is the fastest of these tiles or within 4% of it, but for
// 100000x32x240 (144 on 128 rows, 129 on 64).  The direct loads win from
// K of 160 to 200 on where their rounds are full (6000x6000x224 985 against
// 999; 14400x1920x256 865 against 882), the 64x64 tiles below (16900x1300x100
// 329 against 367), 32 columns where 64 pad more (38000x200x200, batch 3 702
// against 745; 90x90x200, batch 700 256 against 304), 32 rows likewise
// (70x5000x240, batch 20 337 against 409).  Outputs at most 32 wide
// stay on 32 columns (128 rows, 64 if the output has no more).
// The XCD-grouped order re-reads less, but where the result is most of the
// traffic the plain order is ahead (19900x19900x190 9000 against 9379): from
// K = 320 on grouped, and the 64x64 tiles always (8385x8385x45 490 against 520).
static int tile_variant(const GemmArgs& g) {
  if (g.N <= 32) return g.M <= 64 ? GEMM_64x32_G4 : GEMM_128x32_G4_SB;
  const int K = g.kchunk > 0 ? g.kchunk : g.K;
  const double nk = (K + 15) / 16;
  const i64 r64 = (g.M + 63) / 64, r128 = (g.M + 127) / 128, c32 = (g.N + 31) / 32, c64 = (g.N + 63) / 64;
  auto rounds = [&](i64 tiles) { return (double)((tiles * g.batch + 255) / 256); };
  int best = GEMM_64x64_G4_SB_GROUPED;
  double t = rounds(r64 * c64) * (1.98 * nk + 1.0);
  auto offer = [&](int v, double tv) {
    if (tv < t) best = v, t = tv;
  };
  offer(GEMM_128x32_G4_SB, rounds(r128 * c32) * (2.1 * nk + 1.0));
  offer(GEMM_64x32_G4, rounds(r64 * c32) * (1.08 * nk + 1.0));
  // 32 rows, as 32 columns of C^T = B^T A^T; its stores run across the output
  const i64 n64 = (g.N + 63) / 64, n128 = (g.N + 127) / 128, m32 = (g.M + 31) / 32;
  offer(kTransposedChoice + GEMM_128x32_G4_SB, 1.05 * rounds(n128 * m32) * (2.1 * nk + 1.0));
  offer(kTransposedChoice + GEMM_64x32_G4, 1.05 * rounds(n64 * m32) * (1.08 * nk + 1.0));
  offer(K < 320 ? GEMM_128x128_DMA : GEMM_128x128_DMA_GROUPED, dma_cost(g));
  return best;
}

int gemm_by_rule(cclr_ctx* c, const GemmArgs& g) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0 || g.K <= 0) return -1;
  if (frag_may_pay(g)) {
    small_product(c, g);
    return kFormFrag;
  }
  if (even_split(c, g)) return kFormEven;
  const int v = tile_variant(g);
  launch_gemm_choice(g, v, c->stream);
  // the record of large products, one line for each shape (the parts of one
  // that is split along K are none)
  if (g.kchunk == 0 && 8.0 * g.M * (double)g.N * g.K * g.batch >= 1e10 && c->gemm_record.size() < 256)
    c->gemm_record.emplace(std::make_tuple(g.M, g.N, g.K, g.batch), v);
  return v;
}

// -------------------------------------------------------- integral views
Ten fblk(cclr_ctx* c, const char* kinds) {
  const int o = c->o, n = c->o + c->v;
  Ten t = ten(c->f.c(), {(i64)n, (i64)n});
  i64 off = (kinds[0] == 'o' ? 0 : o) * (i64)n + (kinds[1] == 'o' ? 0 : o);
  t.p += off;
  t.dim[0] = kinds[0] == 'o' ? o : c->v;
  t.dim[1] = kinds[1] == 'o' ? o : c->v;
  return t;
}

Ten Vblk(cclr_ctx* c, const char* kinds) {
  const i64 o = c->o, v = c->v;
  auto sz = [&](char k) { return k == 'o' ? o : v; };
  std::string bra(kinds, 2), ket(kinds + 2, 2);
  double sign = 1.0;
  // labels track axis identity: requested axes are "pqrs"
  std::string lab = "pqrs";
  if (bra == "vo") { bra = "ov"; sign = -sign; std::swap(lab[0], lab[1]); }
  if (ket == "vo") { ket = "ov"; sign = -sign; std::swap(lab[2], lab[3]); }
  auto rank = [](const std::string& s) { return s == "oo" ? 0 : (s == "ov" ? 1 : 2); };
  Ten base;
  std::string baselab;
  bool cj = false;
  auto blk = [&](const std::string& k) -> DevBuf& {
    if (k == "oooo") return c->Voooo;
    if (k == "ooov") return c->Vooov;
    if (k == "oovv") return c->Voovv;
    if (k == "ovov") return c->Vovov;
    if (k == "ovvv") return c->Vovvv;
    if (k == "vvvv") return c->Vvvvv;
    throw CclrError(CCLR_EINVAL, "Vblk: no block " + k);
  };
  if (rank(bra) <= rank(ket)) {
    std::string k = bra + ket;
    base = ten(blk(k), {sz(k[0]), sz(k[1]), sz(k[2]), sz(k[3])});
    baselab = lab;  // base axes carry labels lab[0..3]
  } else {
    std::string k = ket + bra;
    base = ten(blk(k), {sz(k[0]), sz(k[1]), sz(k[2]), sz(k[3])});
    // V[pqrs] = conj(Vbase[rspq]): base axes are (r, s, p, q) of the request
    baselab = std::string() + lab[2] + lab[3] + lab[0] + lab[1];
    cj = true;
  }
  Ten r = reorder(base, baselab.c_str(), "pqrs");
  r.conj = cj;
  r.sr = sign;
  r.si = 0.0;
  return r;
}
