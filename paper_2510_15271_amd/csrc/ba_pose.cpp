// Pose-only refinement against a fixed map (paper Sec. 6.4.2, localization
// mode): every request of a call runs in one launch, one workgroup each.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <memory>
#include <new>
#include <system_error>
#include <thread>
#include <vector>

#include "../../include/ba.h"
#include "ba_internal.h"
#include "ba_runtime.h"

namespace bax {

static bool request_sized(const ba_pose_request &r) {
  return r.n >= 1 && r.n <= BA_POSE_MAX_CORR && r.X && r.uv;
}

// Whether every value is finite: adding one to the exponent field carries into the sign
// bit exactly where the field is all ones.
static bool all_finite(const double *v, int64_t n) {
  uint64_t m = 0;
  for (int64_t i = 0; i < n; ++i) {
    uint64_t b;
    std::memcpy(&b, v + i, 8);
    m |= (b & 0x7fffffffffffffffull) + 0x0010000000000000ull;
  }
  return !(m >> 63);
}

// The parts of a request's check before its correspondences.
static int check_pose_head(const ba_pose_request &r, int64_t i) {
  if (r.n < 1 || r.n > BA_POSE_MAX_CORR)
    return fail(BA_EINVAL, "request %lld: n = %d outside [1, %d]", (long long)i, r.n, BA_POSE_MAX_CORR);
  if (!r.X || !r.uv) return fail(BA_EINVAL, "request %lld: NULL correspondence array", (long long)i);
  if (!(std::isfinite(r.K.fx) && std::isfinite(r.K.fy) && std::isfinite(r.K.cx) && std::isfinite(r.K.cy)) ||
      r.K.fx == 0.0 || r.K.fy == 0.0)
    return fail(BA_EINVAL, "request %lld: invalid intrinsics", (long long)i);
  return check_pose(r.pose0, "request", i);
}

int check_pose_request(const ba_pose_request &r, int64_t i) {
  if (int e = check_pose_head(r, i)) return e;
  if (!all_finite(r.X, 3 * (int64_t)r.n))
    return fail(BA_EINVAL, "request %lld: non-finite map point", (long long)i);
  if (!all_finite(r.uv, 2 * (int64_t)r.n)) return fail(BA_EINVAL, "request %lld: non-finite pixel", (long long)i);
  return BA_OK;
}

// Device block of a batch: [PoseDev x n][X double][uv float].
int PoseBatch::lay_out(const std::vector<const ba_pose_request *> &reqs, const std::vector<const ba_options *> &opts) {
  n = (int)reqs.size();
  hdr.assign(n, PoseDev{});
  int64_t o = 0;
  for (int i = 0; i < n; ++i) {
    const ba_pose_request &r = *reqs[i];
    PoseDev &d = hdr[i];
    d.K[0] = r.K.fx;
    d.K[1] = r.K.fy;
    d.K[2] = r.K.cx;
    d.K[3] = r.K.cy;
    quat_to_pose12(r.pose0, d.pose);
    d.off = o;
    d.n = r.n;
    d.iters = opts[i]->max_iters;
    d.delta = opts[i]->huber_delta;
    o += r.n;
  }
  n_corr = o;
  X.reset(new (std::nothrow) double[3 * (size_t)o]);  // (not cleared: written in full)
  uv.reset(new (std::nothrow) float[2 * (size_t)o]);
  if (!X || !uv) return fail(BA_ENOMEM, "no memory to stage %lld correspondences", (long long)o);
  return BA_OK;
}

bool PoseBatch::pack_range(const std::vector<const ba_pose_request *> &reqs, int i0, int i1) {
  bool ok = true;
  for (int i = i0; i < i1; ++i) {
    const ba_pose_request &r = *reqs[i];
    const int64_t o = hdr[i].off;
    ok = ok && all_finite(r.X, 3 * (int64_t)r.n) && all_finite(r.uv, 2 * (int64_t)r.n);
    std::memcpy(&X[3 * o], r.X, 3 * (size_t)r.n * sizeof(double));
    for (int c = 0; c < 2 * r.n; ++c) uv[2 * o + c] = (float)r.uv[c];
  }
  return ok;
}

int PoseBatch::pack(const std::vector<const ba_pose_request *> &reqs, const std::vector<const ba_options *> &opts) {
  if (int e = lay_out(reqs, opts)) return e;
  (void)pack_range(reqs, 0, n);  // (checked by the caller)
  return BA_OK;
}

static size_t up256(size_t b) { return (b + 255) & ~size_t(255); }
double *PoseBatch::dev_X(char *base) const { return (double *)(base + up256((size_t)n * sizeof(PoseDev))); }
float *PoseBatch::dev_uv(char *base) const { return (float *)((char *)dev_X(base) + up256((size_t)n_corr * 3 * 8)); }
size_t PoseBatch::bytes() const {
  return up256((size_t)n * sizeof(PoseDev)) + up256((size_t)n_corr * 3 * 8) + (size_t)n_corr * 2 * 4;
}

int PoseBatch::launch(char *base, hipStream_t s, KernelTimer *tm) {
  PoseDev *dh = (PoseDev *)base;
  hipError_t e = hipMemcpyAsync(dh, hdr.data(), n * sizeof(PoseDev), hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = launch_pose_gn(n, dh, dev_X(base), dev_uv(base), s, tm);
  if (e == hipSuccess) e = hipMemcpyAsync(hdr.data(), dh, n * sizeof(PoseDev), hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return hip_fail(e, "pose batch");
  return BA_OK;
}

int PoseBatch::run(char *base, hipStream_t s, KernelTimer *tm) {
  hipError_t e = hipMemcpyAsync(dev_X(base), X.get(), (size_t)n_corr * 3 * 8, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipMemcpyAsync(dev_uv(base), uv.get(), (size_t)n_corr * 2 * 4, hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return hip_fail(e, "pose batch");
  return launch(base, s, tm);
}

// Checks, packs and uploads a batch's correspondences in blocks of about kBlockCorr: the
// blocks are packed by up to kPackThreads threads (this one among them) while the finished
// ones are uploaded in order by this thread, which makes every HIP call.  bad: the first
// request with a value that is not finite, or n.  Staging them in one thread, then copying,
// took most of a large call (4096 requests, 2.6 M correspondences: 69 ms with the requests'
// marshalling, 14.5 so).
constexpr int64_t kBlockCorr = 1 << 16;
constexpr int kPackThreads = 8;
static int pack_and_upload(PoseBatch &pb, const std::vector<const ba_pose_request *> &reqs, char *base, hipStream_t s,
                           int &bad) {
  std::vector<int> cut{0};  // first request of each block, then n
  for (int i = 0; i < pb.n; ++i)
    if (pb.hdr[i].off - pb.hdr[cut.back()].off >= kBlockCorr) cut.push_back(i);
  cut.push_back(pb.n);
  const int nb = (int)cut.size() - 1;
  std::unique_ptr<std::atomic<int>[]> done(new std::atomic<int>[nb]);  // 0: open, 1: packed, 2: not finite
  for (int b = 0; b < nb; ++b) done[b] = 0;
  std::atomic<int> next{0};
  auto pack_one = [&] {
    const int b = next++;
    if (b >= nb) return false;
    done[b].store(pb.pack_range(reqs, cut[b], cut[b + 1]) ? 1 : 2, std::memory_order_release);
    return true;
  };
  std::vector<std::thread> th;
  const int nt = std::min({kPackThreads, nb, (int)std::max(1u, std::thread::hardware_concurrency())});
  try {
    for (int x = 1; x < nt; ++x)
      th.emplace_back([&] {
        while (pack_one()) {
        }
      });
  } catch (const std::system_error &) {  // fewer threads: the others pack all the same
  }
  hipError_t e = hipSuccess;
  bad = pb.n;
  for (int b = 0; b < nb; ++b) {
    int st;
    while (!(st = done[b].load(std::memory_order_acquire)))
      if (!pack_one()) std::this_thread::yield();
    if (st == 2 && bad == pb.n)
      for (int i = cut[b]; i < cut[b + 1] && bad == pb.n; ++i)
        if (!all_finite(reqs[i]->X, 3 * (int64_t)reqs[i]->n) || !all_finite(reqs[i]->uv, 2 * (int64_t)reqs[i]->n)) bad = i;
    if (bad < pb.n || e != hipSuccess) continue;  // only wait for the threads
    const int64_t o = pb.hdr[cut[b]].off, m = (cut[b + 1] < pb.n ? pb.hdr[cut[b + 1]].off : pb.n_corr) - o;
    e = hipMemcpyAsync(pb.dev_X(base) + 3 * o, &pb.X[3 * o], (size_t)m * 3 * 8, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
      e = hipMemcpyAsync(pb.dev_uv(base) + 2 * o, &pb.uv[2 * o], (size_t)m * 2 * 4, hipMemcpyHostToDevice, s);
  }
  for (std::thread &t : th) t.join();
  return e == hipSuccess ? BA_OK : hip_fail(e, "pose batch");
}

}  // namespace bax

using namespace bax;

extern "C" int ba_pose_batch(int32_t n_req, const ba_pose_request *reqs, const ba_options *opt,
                             void *hip_stream, ba_pose *poses_out, int32_t *status_out,
                             double *cost_out, double *device_ms) {
  if (n_req < 1 || !reqs) return fail(BA_EINVAL, "no requests");
  if (int e = check_options(opt, true)) return e;
  std::vector<const ba_pose_request *> rp(n_req);
  for (int i = 0; i < n_req; ++i) {
    // the first request that fails is reported: those before it have their values checked too
    if (!request_sized(reqs[i]) || check_pose_head(reqs[i], i)) {
      for (int k = 0; k <= i; ++k)
        if (int e = check_pose_request(reqs[k], k)) return e;
    }
    rp[i] = &reqs[i];
  }
  PoseBatch pb;
  if (int e = pb.lay_out(rp, std::vector<const ba_options *>(n_req, opt))) return e;
  hipStream_t s = (hipStream_t)hip_stream;
  bool own = false;
  hipError_t e = hipSuccess;
  // a device error is reported only for requests that are valid
  auto device_error = [&](hipError_t err, const char *what) {
    for (int i = 0; i < n_req; ++i)
      if (int r = check_pose_request(reqs[i], i)) return r;
    return hip_fail(err, what);
  };
  if (!s) {
    e = hipStreamCreate(&s);
    if (e != hipSuccess) return device_error(e, "hipStreamCreate");
    own = true;
  }
  void *mem = nullptr;
  e = hipMalloc(&mem, pb.bytes());
  if (e != hipSuccess) {
    if (own) (void)hipStreamDestroy(s);
    return device_error(e, "pose batch allocation");
  }
  EventTimer timer;  // device time of the pose kernel alone
  int bad = n_req;
  int rc = pack_and_upload(pb, rp, (char *)mem, s, bad);
  if (rc == BA_OK && bad == n_req) rc = pb.launch((char *)mem, s, &timer);
  // (also after an error: the copies that were queued read the staging arrays)
  e = hipStreamSynchronize(s);
  if (rc == BA_OK && e != hipSuccess) rc = hip_fail(e, "pose batch");
  if (rc == BA_OK && bad < n_req) rc = check_pose_request(reqs[bad], bad);
  if (rc == BA_OK) {
    double ms[K_NUM_KERNELS];
    int32_t nl[K_NUM_KERNELS];
    timer.collect(ms, nl);
    if (device_ms) *device_ms = ms[K_POSE_GN];
    for (int i = 0; i < n_req; ++i) {
      if (poses_out) poses_out[i] = pose12_to_quat(pb.hdr[i].pose);
      if (status_out) status_out[i] = pb.hdr[i].status;
      if (cost_out) cost_out[i] = pb.hdr[i].cost;
    }
  }
  (void)hipFree(mem);
  if (own) (void)hipStreamDestroy(s);
  return rc;
}
