// Rows from the device to the caller's ordinary (pageable) memory.
//
// The runtime's copy to pageable memory runs at 11 to 17 GB/s; one to pinned memory
// at 55, and one core then moves 30 (out of its caches) to 70 GB/s.  So the rows go
// through two pinned pieces, the copy of one piece running while the core
// empties the other.  A call with its copy, before and now: 37 rows of 100,003
// nodes (14.8 MB) 990 and 660 us, 512 of 65,536 (134 MB) 12.3 and 4.9 ms.  Below
// kDirectBytes there is little to gain (1.2 MB 97 and 91 us, 0.5 MB 53 and 66) for
// the 0.5 to 1 ms that pinning the pieces takes once per context.  Pieces of 512 KB,
// 1 and 2 MB took 720, 530 and 430 us for 14.8 MB, as each copy costs 15 us besides;
// four cores instead of one gain nothing there.
#include <string.h>

#include <algorithm>

#include "internal.hpp"

namespace dawn {

namespace {

constexpr size_t kDirectBytes = 8 << 20;
constexpr size_t kPieceBytes = 2 << 20;        // most bytes of a piece
constexpr int kMaxBounces = 4;            // pinned buffers a context holds, taken or not

}  // namespace

// Two pinned pieces and the events of the copies into them.
struct Bounce {
  char* p = nullptr;
  size_t piece = 0;
  hipEvent_t ev[2] = {nullptr, nullptr};
};

static void bounce_free(Bounce* b) {
  if (!b) return;
  for (hipEvent_t e : b->ev)
    if (e) hipEventDestroy(e);
  if (b->p) hipHostFree(b->p);
  delete b;
}

// A buffer with pieces of at least `piece` bytes (null: none to be had).
static Bounce* bounce_take(Ctx* ctx, size_t piece) {
  Bounce* small = nullptr;
  {
    std::lock_guard<std::mutex> lk(ctx->bounce_mu);
    for (size_t i = 0; i < ctx->bounces.size(); ++i)
      if (ctx->bounces[i]->piece >= piece) {
        Bounce* b = ctx->bounces[i];
        ctx->bounces.erase(ctx->bounces.begin() + (long)i);
        return b;
      }
    if (ctx->bounce_count == kMaxBounces) {
      if (ctx->bounces.empty()) return nullptr;
      small = ctx->bounces.back();      // makes way for a larger one
      ctx->bounces.pop_back();
    } else {
      ++ctx->bounce_count;
    }
  }
  bounce_free(small);
  Bounce* b = new Bounce();
  b->piece = piece;
  hipError_t e = hipHostMalloc((void**)&b->p, 2 * piece, hipHostMallocDefault);
  for (hipEvent_t& x : b->ev)
    if (e == hipSuccess) e = hipEventCreateWithFlags(&x, hipEventDisableTiming);
  if (e == hipSuccess) return b;
  (void)hipGetLastError();
  bounce_free(b);
  std::lock_guard<std::mutex> lk(ctx->bounce_mu);
  --ctx->bounce_count;
  return nullptr;
}

static void bounce_give(Ctx* ctx, Bounce* b) {
  std::lock_guard<std::mutex> lk(ctx->bounce_mu);
  ctx->bounces.push_back(b);
}

void bounces_free(Ctx* ctx) {
  std::lock_guard<std::mutex> lk(ctx->bounce_mu);
  for (Bounce* b : ctx->bounces) bounce_free(b);
  ctx->bounces.clear();
  ctx->bounce_count = 0;
}

// Ordinary memory, which the runtime knows nothing of.
static bool pageable(const void* p) {
  hipPointerAttribute_t a;
  if (hipPointerGetAttributes(&a, p) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return a.type == hipMemoryTypeUnregistered;
}

hipError_t copy_rows_to_host(Ctx* ctx, int32_t* dst, size_t dst_stride, const int32_t* src,
                             size_t n, size_t rows, hipStream_t s) {
  size_t row = n * 4, stride = dst_stride * 4;
  if (stride == row) {
    row *= rows;
    stride = row;
    rows = 1;
  }
  const size_t total = row * rows;
  if (total == 0) return hipStreamSynchronize(s);
  Bounce* b = nullptr;
  if (total >= kDirectBytes && pageable(dst)) {
    size_t piece = 64 << 10;
    while (piece < kPieceBytes && 2 * piece < total) piece *= 2;
    b = bounce_take(ctx, piece);
  }
  if (!b) {
    hipError_t e = rows == 1 ? hipMemcpyAsync(dst, src, row, hipMemcpyDeviceToHost, s)
                             : hipMemcpy2DAsync(dst, stride, src, row, row, rows,
                                                hipMemcpyDeviceToHost, s);
    return e == hipSuccess ? hipStreamSynchronize(s) : e;
  }
  const size_t piece = std::min(b->piece, kPieceBytes);
  const size_t pieces = (total + piece - 1) / piece;
  auto start = [&](size_t i) {
    const size_t o = i * piece;
    hipError_t e = hipMemcpyAsync(b->p + (i & 1) * b->piece, (const char*)src + o,
                                  std::min(piece, total - o), hipMemcpyDeviceToHost, s);
    return e == hipSuccess ? hipEventRecord(b->ev[i & 1], s) : e;
  };
  hipError_t e = start(0);
  if (e == hipSuccess && pieces > 1) e = start(1);
  for (size_t i = 0; i < pieces && e == hipSuccess; ++i) {
    e = hipEventSynchronize(b->ev[i & 1]);
    if (e != hipSuccess) break;
    const char* from = b->p + (i & 1) * b->piece;
    size_t o = i * piece;
    const size_t end = std::min(o + piece, total);
    while (o < end) {
      const size_t r = o / row, at = o % row, len = std::min(end - o, row - at);
      memcpy((char*)dst + r * stride + at, from, len);
      from += len;
      o += len;
    }
    if (i + 2 < pieces) e = start(i + 2);
  }
  if (e != hipSuccess) hipStreamSynchronize(s);   // nothing may still write to the pieces
  bounce_give(ctx, b);
  return e;
}

}  // namespace dawn
