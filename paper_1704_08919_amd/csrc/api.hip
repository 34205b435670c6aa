// C ABI of libpairopt.so: argument validation, per-pulse descriptors, scratch management and
// the sequencing of the synthesis, evolution, reduction and differential-evolution kernels.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <mutex>
#include <utility>
#include <cstdio>
#include <cstring>
#include <vector>

#include "common.hpp"

namespace po {

static thread_local std::string g_error;

po_status set_error(po_status s, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_error = buf;
  return s;
}

po_status device_error(hipError_t e, const char* what) {
  (void)hipGetLastError();
  return set_error(e == hipErrorOutOfMemory ? PO_ERR_NOMEM : PO_ERR_DEVICE, "%s failed: %s", what,
                   hipGetErrorString(e));
}

po_status check_device_range(const void* p, size_t bytes, size_t align, const char* name) {
  if (!p) return set_error(PO_ERR_INVALID, "%s is NULL", name);
  if (reinterpret_cast<uintptr_t>(p) % align) return set_error(PO_ERR_INVALID, "%s is not %zu-byte aligned", name, align);
  hipPointerAttribute_t attr;
  std::memset(&attr, 0, sizeof attr);
  hipError_t e = hipPointerGetAttributes(&attr, p);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return set_error(PO_ERR_INVALID, "%s is not a device pointer (%s)", name, hipGetErrorString(e));
  }
  if (attr.type != hipMemoryTypeDevice && attr.type != hipMemoryTypeManaged)
    return set_error(PO_ERR_INVALID, "%s is not device memory (type %d)", name, int(attr.type));
  int dev = -1;
  PO_HIP(hipGetDevice(&dev));
  if (attr.type == hipMemoryTypeDevice && attr.device != dev)
    return set_error(PO_ERR_INVALID, "%s lives on device %d, current device is %d", name, attr.device, dev);
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  e = hipMemGetAddressRange(&base, &size, const_cast<void*>(p));
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return set_error(PO_ERR_INVALID, "%s: allocation range unknown (%s)", name, hipGetErrorString(e));
  }
  const uintptr_t lo = reinterpret_cast<uintptr_t>(base), q = reinterpret_cast<uintptr_t>(p);
  if (q < lo || q - lo > size || bytes > size - (q - lo))
    return set_error(PO_ERR_INVALID, "%s: %zu bytes needed, allocation holds %zu from this pointer", name, bytes,
                     size_t(lo + size - q));
  return PO_OK;
}

namespace {

// One memory pool per device for the calls' scratch.  The device's default pool hands everything back
// at each synchronisation, so a call after one pays for mapping its scratch again (an evaluation with
// 100 MB of it took 1.2 ms, 0.12 ms with the memory kept).  This pool keeps up to kPoolKeep bytes and
// hands back what is beyond; all of it when an allocation fails for lack of memory.  The pool's
// reuse is stream-ordered: memory freed on one stream serves another only behind its work.
constexpr uint64_t kPoolKeep = uint64_t(512) << 20;
constexpr int kMaxDevices = 64;
std::mutex g_pool_mu;
hipMemPool_t g_pool[kMaxDevices] = {};

// The pool cannot be created while a stream of the process is being captured (in the global mode): a call
// that comes first at that time takes its scratch from the device's default pool.
po_status scratch_pool(hipStream_t s, hipMemPool_t* out) {
  int dev = -1;
  PO_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return set_error(PO_ERR_UNSUPPORTED, "device %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_pool_mu);
  if (!g_pool[dev]) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    PO_HIP(hipStreamIsCapturing(s, &cap));
    hipMemPool_t pool = nullptr;
    hipError_t e = hipErrorStreamCaptureUnsupported;
    if (cap == hipStreamCaptureStatusNone) {
      hipMemPoolProps props;
      std::memset(&props, 0, sizeof props);
      props.allocType = hipMemAllocationTypePinned;
      props.location.type = hipMemLocationTypeDevice;
      props.location.id = dev;
      e = hipMemPoolCreate(&pool, &props);
    }
    if (e == hipErrorStreamCaptureUnsupported) {
      (void)hipGetLastError();
      PO_HIP(hipDeviceGetDefaultMemPool(out, dev));
      return PO_OK;
    }
    if (e != hipSuccess) return device_error(e, "hipMemPoolCreate");
    uint64_t keep = kPoolKeep;
    e = hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep);
    if (e != hipSuccess) {
      (void)hipMemPoolDestroy(pool);
      return device_error(e, "hipMemPoolSetAttribute");
    }
    g_pool[dev] = pool;
  }
  *out = g_pool[dev];
  return PO_OK;
}

}  // namespace

po_status Scratch::alloc(size_t bytes, hipStream_t s) {
  stream = s;
  if (bytes == 0) bytes = 8;
  hipMemPool_t pool = nullptr;
  PO_TRY(scratch_pool(s, &pool));
  hipError_t e = hipMallocFromPoolAsync(&ptr, bytes, pool, s);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    (void)hipMemPoolTrimTo(pool, 0);
    e = hipMallocFromPoolAsync(&ptr, bytes, pool, s);
  }
  if (e != hipSuccess) {
    ptr = nullptr;
    return device_error(e, "hipMallocFromPoolAsync");
  }
  return PO_OK;
}

po_status validate_spec(const po_pulse_spec& s, int i) {
  if (!(s.T > 0.0) || !std::isfinite(s.T)) return set_error(PO_ERR_INVALID, "spec %d: T must be finite and > 0", i);
  if (s.nt < 2 || s.nt > (1 << 24)) return set_error(PO_ERR_INVALID, "spec %d: nt must be in [2, 2^24]", i);
  if (s.order < 1 || s.n_s < s.order || s.n_s > kMaxNs)
    return set_error(PO_ERR_INVALID, "spec %d: need 1 <= order <= n_s <= %d", i, kMaxNs);
  if (!(s.omega_min >= 0.0) || !(s.omega_max > s.omega_min) || !std::isfinite(s.omega_max))
    return set_error(PO_ERR_INVALID, "spec %d: need 0 <= omega_min < omega_max", i);
  const double dw = 2.0 * M_PI / s.T;
  const double r = s.omega_min / dw;
  if (std::fabs(r - std::nearbyint(r)) > 1e-9) return set_error(PO_ERR_INVALID, "spec %d: omega_min / (2 pi / T) must be an integer", i);
  const double nl = std::floor((s.omega_max - s.omega_min) / dw + 1e-9) + 1.0;
  if (nl > kMaxLines) return set_error(PO_ERR_INVALID, "spec %d: %g spectral lines exceed %d", i, nl, kMaxLines);
  if (s.norm != PO_NORM_NONE && s.norm != PO_NORM_PEAK && s.norm != PO_NORM_ENERGY)
    return set_error(PO_ERR_INVALID, "spec %d: unknown norm %d", i, s.norm);
  if (s.norm != PO_NORM_NONE && !(s.norm_value > 0.0 && std::isfinite(s.norm_value)))
    return set_error(PO_ERR_INVALID, "spec %d: norm_value must be finite and > 0", i);
  return PO_OK;
}

po_status validate_grid(const po_grid& g, int i) {
  for (int d = 0; d < 3; ++d) {
    if (g.n[d] < 1) return set_error(PO_ERR_INVALID, "grid %d: n[%d] must be >= 1", i, d);
    if (!std::isfinite(g.lo[d]) || !std::isfinite(g.hi[d]) || g.lo[d] > g.hi[d])
      return set_error(PO_ERR_INVALID, "grid %d: need finite lo[%d] <= hi[%d]", i, d, d);
    if (g.n[d] > 1 && !(g.lo[d] < g.hi[d])) return set_error(PO_ERR_INVALID, "grid %d: n[%d] > 1 needs lo < hi", i, d);
  }
  const int64_t m = int64_t(g.n[0]) * g.n[1] * g.n[2];
  if (m > (int64_t(1) << 30)) return set_error(PO_ERR_INVALID, "grid %d: more than 2^30 modes", i);
  return PO_OK;
}

po_status build_batch(int32_t n, const po_pulse_spec* specs, const po_grid* grids, PulseDev* out, Batch* b) {
  *b = Batch{};
  b->n_pulses = n;
  int64_t tab = 0, modes = 0, coeff = 0, spec = 0;
  int64_t units = 0, items = 0, chunks = 0, lines = 0, harm = 0;
  for (int i = 0; i < n; ++i) {
    PulseDev d;
    std::memset(&d, 0, sizeof d);
    d.tab_off = tab;
    d.mode_off = modes;
    d.coeff_off = coeff;
    d.spec_off = spec;
    d.line_off = lines;
    d.harm_off = harm;
    d.unit_off = units;
    d.item_off = int32_t(items);
    d.chk_off = int32_t(chunks);
    if (specs) {
      const po_pulse_spec& s = specs[i];
      d.nt = s.nt;
      d.ns = s.n_s;
      d.order = s.order;
      d.T = s.T;
      d.dt = s.T / double(s.nt);
      d.dw = 2.0 * M_PI / s.T;
      d.wmin = s.omega_min;
      d.wmax = s.omega_max;
      d.nmin = int32_t(std::nearbyint(s.omega_min / d.dw));
      d.nlines = int32_t(std::floor((s.omega_max - s.omega_min) / d.dw + 1e-9)) + 1;
      d.norm = s.norm;
      d.norm_value = s.norm_value;
      d.stat_blocks =
          s.norm == PO_NORM_NONE ? 0 : (image_bases(s.nt, s.norm == PO_NORM_PEAK ? s.nt : s.nt - 1) + 255) / 256;
      b->max_bases = std::max(b->max_bases, image_bases(s.nt, s.nt - 1));
      tab += s.nt;
      chunks += (s.nt + kChunkSteps - 1) / kChunkSteps;
      coeff += 4 * int64_t(s.n_s);
      spec += kSpecRec * (int64_t(spec_records(d.nlines)) + 1);
      lines += d.nlines;
      harm += d.nlines + 2;
      b->max_nt = std::max(b->max_nt, s.nt);
      b->max_lines = std::max(b->max_lines, d.nlines);
      b->max_ns = std::max(b->max_ns, d.ns);
      b->max_stat_blocks = std::max(b->max_stat_blocks, d.stat_blocks);
    }
    if (grids) {
      const po_grid& g = grids[i];
      double dv = 1.0;
      for (int k = 0; k < 3; ++k) {
        d.n[k] = g.n[k];
        d.lo[k] = g.lo[k];
        const bool sheet = g.n[k] == 1 && g.lo[k] == g.hi[k];
        d.dp[k] = sheet ? 0.0 : (g.hi[k] - g.lo[k]) / double(g.n[k]);
        if (!sheet) dv *= d.dp[k];
      }
      d.dv = dv;
      const int64_t m = int64_t(g.n[0]) * g.n[1] * g.n[2];
      d.mirror = g.n[2] > 1 && g.lo[2] == -g.hi[2] ? 1 : 0;
      d.ndist = d.mirror ? int64_t(g.n[0]) * g.n[1] * ((g.n[2] + 1) / 2) : m;
      if (kItem % g.n[0] != 0 || int64_t(g.n[0]) * g.n[1] % (2 * kItem) != 0) b->row_pairs = false;
      d.nunits = int32_t((d.ndist + kUnit - 1) / kUnit);
      d.nitems = int32_t((d.ndist + kItem - 1) / kItem);
      b->total_units_all += (m + kUnit - 1) / kUnit;
      modes += m;
      units += d.nunits;
      items += d.nitems;
    }
    out[i] = d;
  }
  if (items > (int64_t(1) << 31) - 1) return set_error(PO_ERR_INVALID, "batch has too many modes");
  int64_t slots = 0, part = 0;
  if (specs && grids)
    for (int i = 0; i < n; ++i) {
      // Few modes leave the chip idle along the mode axis, so they get more segments: 128 slots for a
      // 1024-mode sheet (62 us for the whole evaluation at nt = 4096; 67 us with 16 or 64 segments, the
      // latter spent on applying them), 8 segments from 16384 modes on, where a batch of any size fills
      // the chip and each further segment only costs its product with the state.  A matter of the
      // pulse's own sizes: its result does not depend on the batch.
      int want = 8;
      while (want < 32 && want * out[i].nitems < 512) want *= 2;
      const int units = (out[i].nt + kSegUnit - 1) / kSegUnit;
      out[i].seg_len = (units + want - 1) / want * kSegUnit;
      out[i].nseg = (out[i].nt + out[i].seg_len - 1) / out[i].seg_len;
      out[i].slot_off = slots;
      slots += int64_t(out[i].nitems) * out[i].nseg;
      out[i].part_off = 2 * part;
      part += int64_t(out[i].nitems) * out[i].nt;
    }
  b->total_slots = slots;
  b->total_rows = tab;
  b->total_modes = modes;
  b->total_coeff = coeff;
  b->total_spec = spec;
  b->total_lines = lines;
  b->total_harm = harm;
  b->total_units = units;
  b->total_items = int32_t(items);
  b->total_chunks = int32_t(chunks);
  return PO_OK;
}

namespace {

po_status check_specs(int32_t n, const po_pulse_spec* specs) {
  if (!specs) return set_error(PO_ERR_INVALID, "specs is NULL");
  for (int i = 0; i < n; ++i) PO_TRY(validate_spec(specs[i], i));
  return PO_OK;
}

po_status check_grids(int32_t n, const po_grid* grids) {
  if (!grids) return set_error(PO_ERR_INVALID, "grids is NULL");
  for (int i = 0; i < n; ++i) PO_TRY(validate_grid(grids[i], i));
  return PO_OK;
}

// Descriptors of a few pulses as a kernel argument.
constexpr int kArgPulses = 8;
struct DescPack {
  PulseDev d[kArgPulses];
};

__global__ void __launch_bounds__(64) k_put_desc(DescPack p, int n, PulseDev* __restrict__ out) {
  for (int i = threadIdx.x; i < n; i += 64) out[i] = p.d[i];
}

// Descriptors of n pulses alike: pulse 0's, with the offsets of pulse i at i times pulse 1's.
__global__ void __launch_bounds__(64) k_fill_desc(PulseDev d, PulseDev step, int n, PulseDev* __restrict__ out) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i >= n) return;
  d.tab_off = i * step.tab_off;
  d.mode_off = i * step.mode_off;
  d.coeff_off = i * step.coeff_off;
  d.spec_off = i * step.spec_off;
  d.line_off = i * step.line_off;
  d.harm_off = i * step.harm_off;
  d.chk_off = i * step.chk_off;
  d.unit_off = i * step.unit_off;
  d.item_off = i * step.item_off;
  d.slot_off = i * step.slot_off;
  d.part_off = i * step.part_off;
  out[i] = d;
}

// Puts the descriptors into device memory: by kernel arguments where they fit (a few pulses, or pulses
// alike), which spares the copy from pageable host memory (it takes longer than these kernels, and
// the host waits for it), else by that copy.  Under capture always by kernel arguments, a few at a time: a recorded copy
// would read the host's array at the replay, when it is gone.
po_status put_desc(const std::vector<PulseDev>& h, PulseDev* d_desc, hipStream_t s) {
  static_assert(sizeof(DescPack) <= 3840, "kernel arguments are limited to 4 KiB");
  const int n = int(h.size());
  const auto put_few = [&](int first) -> po_status {
    const int few = std::min(kArgPulses, n - first);
    DescPack p;
    std::memcpy(p.d, h.data() + first, sizeof(PulseDev) * size_t(few));
    for (int i = few; i < kArgPulses; ++i) std::memset(&p.d[i], 0, sizeof(PulseDev));
    hipLaunchKernelGGL(k_put_desc, dim3(1), dim3(64), 0, s, p, few, d_desc + first);
    PO_HIP(hipGetLastError());
    return PO_OK;
  };
  if (n <= kArgPulses) return put_few(0);
  bool alike = true;
  for (int i = 2; i < n && alike; ++i) {
    PulseDev e;
    std::memcpy(&e, &h[0], sizeof e);
    const PulseDev& u = h[1];
    e.tab_off = i * u.tab_off;
    e.mode_off = i * u.mode_off;
    e.coeff_off = i * u.coeff_off;
    e.spec_off = i * u.spec_off;
    e.line_off = i * u.line_off;
    e.harm_off = i * u.harm_off;
    e.chk_off = i * u.chk_off;
    e.unit_off = i * u.unit_off;
    e.item_off = i * u.item_off;
    e.slot_off = i * u.slot_off;
    e.part_off = i * u.part_off;
    alike = std::memcmp(&e, &h[i], sizeof e) == 0;
  }
  if (alike) {
    PulseDev e;
    std::memcpy(&e, &h[1], sizeof e);
    e.tab_off = e.mode_off = e.coeff_off = e.spec_off = e.line_off = e.harm_off = e.unit_off = e.slot_off = e.part_off = 0;
    e.chk_off = e.item_off = 0;
    alike = std::memcmp(&e, &h[0], sizeof e) == 0;
  }
  if (alike) {
    hipLaunchKernelGGL(k_fill_desc, dim3((n + 63) / 64), dim3(64), 0, s, h[0], h[1], n, d_desc);
    PO_HIP(hipGetLastError());
    return PO_OK;
  }
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  PO_HIP(hipStreamIsCapturing(s, &cap));
  if (cap != hipStreamCaptureStatusNone) {
    for (int i = 0; i < n; i += kArgPulses) PO_TRY(put_few(i));
    return PO_OK;
  }
  PO_HIP(hipMemcpyAsync(d_desc, h.data(), sizeof(PulseDev) * h.size(), hipMemcpyHostToDevice, s));
  return PO_OK;
}

// Scratch of one evaluation (synthesis + evolution + yield), in elements (units: as if no grid were
// mirror-symmetric, which keeps the allocation-free path's limit a matter of the grid's size).
struct EvalSizes {
  size_t spec, part, scl, units, ranges;
};

EvalSizes eval_sizes(int32_t n, const Batch& b) {
  return EvalSizes{size_t(b.total_spec), size_t(std::max(1, b.max_stat_blocks)) * n, size_t(n),
                   size_t(b.total_units_all), 4 * size_t(b.total_chunks)};
}

// Work buffers of the parts of a call: descriptors, synthesis, evolution (in the form the batch takes).
struct DescWork {
  size_t desc;
  DescWork(Work& w, int32_t n) : desc(w.add(sizeof(PulseDev) * n)) {}
};
struct SynthWork {
  size_t spec, part, scl;
  SynthWork(Work& w, int32_t n, const Batch& b) {
    const EvalSizes z = eval_sizes(n, b);
    spec = w.add(sizeof(double) * z.spec);
    part = w.add(sizeof(double) * z.part);
    scl = w.add(sizeof(double) * z.scl);
  }
};
struct AdjointWork {  // tables of the pulses and the line terms of the synthesis adjoint
  size_t A, E, edge, scale, harm, lines;
  AdjointWork(Work& w, int32_t n, const Batch& b) {
    A = w.add(sizeof(double) * 2 * size_t(b.total_rows));
    E = w.add(sizeof(double) * 2 * size_t(b.total_rows));
    edge = w.add(sizeof(double) * 4 * n);
    scale = w.add(sizeof(double) * n);
    harm = w.add(sizeof(double) * 8 * size_t(b.total_harm));
    lines = w.add(sizeof(double) * size_t(b.total_lines) * (8 + size_t(b.max_ns)));
  }
};
struct EvolveWork {
  size_t units, ranges, prop;
  bool split;
  EvolveWork(Work& w, const Batch& b) : split(split_in_time(b)) {
    units = w.add(sizeof(double) * size_t(b.total_units));
    ranges = w.add(sizeof(double) * 4 * size_t(b.total_chunks));
    prop = split ? w.add(sizeof(double) * kSlotDoubles * size_t(b.total_slots)) : 0;
  }
};

po_status synth_impl(const Work& w, const SynthWork& z, const double* d_coeff, double* d_A, double* d_E,
                     double* d_A_edge, double* d_scale, double* d_ranges, hipStream_t s, const Batch& b,
                     const PulseDev* d_desc) {
  return launch_synth(b, d_desc, d_coeff, w.at<double>(z.spec), w.at<double>(z.part), w.at<double>(z.scl), d_A, d_E,
                      d_A_edge, d_scale, d_ranges, s);
}

// Event pairs bracketing evolution launches while timers are enabled.
std::mutex g_timer_mu;
bool g_timer_on = false;
std::vector<std::pair<hipEvent_t, hipEvent_t>> g_timer_events;
unsigned long long* g_counts = nullptr;  // device: mode-steps per series variant (diagnostics)

// Evolution and yield into caller-provided scratch: d_units [total_units] (used when d_J is
// non-NULL), d_ranges [4 total_chunks].  timed: bracket the evolution with the kernel timers.
// d_prop: scratch of the time-split form, or NULL for the form without; have_ranges: the synthesis has
// already written d_ranges.
po_status evolve_into(const Batch& b, const PulseDev* d_desc, const double* d_A, const double* d_A_edge, double* d_f,
                      double* d_J, hipStream_t s, double* d_units, double* d_ranges, bool have_ranges, double* d_prop,
                      bool timed_ok) {
  hipEvent_t e0 = nullptr;
  const bool timed = timed_ok && timer_start(s, &e0);
  if (!have_ranges) PO_TRY(launch_chunk_ranges(b, d_desc, d_A, d_ranges, s));
  double* units = d_J ? d_units : nullptr;
  if (d_prop) PO_TRY(launch_evolve_segments(b, d_desc, d_A, d_A_edge, d_ranges, d_prop, d_f, units, s));
  else PO_TRY(launch_evolve_grid(b, d_desc, d_A, d_A_edge, d_ranges, d_f, units, s));
  if (timed) {
    timer_stop(s, e0);
    PO_TRY(timer_count(b.n_pulses, d_desc, d_ranges, s));
  }
  if (d_J) PO_TRY(launch_yield_from_units(b, d_desc, d_units, d_J, s));
  return PO_OK;
}

po_status evolve_impl(const Work& w, const EvolveWork& z, const Batch& b, const PulseDev* d_desc, const double* d_A,
                      const double* d_A_edge, bool have_ranges, double* d_f, double* d_J, hipStream_t s) {
  return evolve_into(b, d_desc, d_A, d_A_edge, d_f, d_J, s, w.at<double>(z.units), w.at<double>(z.ranges), have_ranges,
                     z.split ? w.at<double>(z.prop) : nullptr, true);
}

// Gradient of J with respect to the tables (forward and adjoint sweeps per mode, fixed-order sums).
// The items are taken in groups whose segment propagators and partial sums stay within kGradGroup bytes, one
// after the other in the same buffers: as many whole pulses as fit, or a part of one that does not.
constexpr int64_t kGradGroup = int64_t(2) << 30;

struct GradWork {
  size_t prop, part, epart, units, ranges;
  std::vector<GradRange> groups;
  GradWork(Work& w, const std::vector<PulseDev>& h, const Batch& b) {
    int64_t max_slots = 0, max_rows = 0, max_items = 0;
    const auto item_bytes = [](const PulseDev& d) {
      return d.nseg * int64_t(sizeof(double)) * kSlotDoubles + 16 * int64_t(d.nt) + 128;
    };
    for (int i = 0, li = 0; i < b.n_pulses;) {  // next item: li of pulse i
      const PulseDev& f = h[i];
      GradRange r{i, i, f.slot_off + int64_t(li) * f.nseg, 0, f.part_off + 2 * int64_t(li) * f.nt, f.item_off + li, 0, 0};
      int64_t rows = 0, left = kGradGroup;
      while (r.i1 < b.n_pulses) {
        const PulseDev& d = h[r.i1];
        const int64_t fit = left / item_bytes(d), rest = d.nitems - li;
        if (r.items > 0 && rest > fit) break;
        const int64_t take = std::min(rest, std::max<int64_t>(fit, 1));
        left -= take * item_bytes(d);
        r.slots += take * d.nseg;
        rows += take * d.nt;
        r.items += int(take);
        r.max_nt = std::max(r.max_nt, d.nt);
        ++r.i1;
        li = take < rest ? li + int(take) : 0;
        if (li > 0) break;
      }
      max_slots = std::max(max_slots, r.slots);
      max_rows = std::max(max_rows, rows);
      max_items = std::max<int64_t>(max_items, r.items);
      groups.push_back(r);
      i = li > 0 ? r.i1 - 1 : r.i1;
    }
    prop = w.add(sizeof(double) * kSlotDoubles * size_t(max_slots));
    part = w.add(sizeof(double) * 2 * size_t(max_rows));
    epart = w.add(sizeof(double) * 16 * size_t(max_items));
    units = w.add(sizeof(double) * size_t(b.total_units));
    ranges = w.add(sizeof(double) * 4 * size_t(b.total_chunks));
  }
};

po_status yield_grad_impl(const Work& w, const GradWork& z, const Batch& b, const PulseDev* d_desc, const double* d_A,
                          const double* d_A_edge, bool have_ranges, double* d_J, double* d_gA, double* d_gedge,
                          hipStream_t s) {
  if (!have_ranges) PO_TRY(launch_chunk_ranges(b, d_desc, d_A, w.at<double>(z.ranges), s));
  for (const GradRange& r : z.groups)
    PO_TRY(launch_yield_grad(d_desc, r, d_A, d_A_edge, w.at<double>(z.ranges), w.at<double>(z.prop),
                             w.at<double>(z.part), w.at<double>(z.epart), w.at<double>(z.units), d_gA, d_gedge, s));
  if (d_J) PO_TRY(launch_yield_from_units(b, d_desc, w.at<double>(z.units), d_J, s));
  return PO_OK;
}

po_status check_differentiable(int32_t n, const po_pulse_spec* specs) {
  for (int i = 0; i < n; ++i)
    if (specs[i].norm == PO_NORM_PEAK)
      return set_error(PO_ERR_UNSUPPORTED, "spec %d: the peak normalisation is not differentiable; use "
                                           "PO_NORM_NONE (with an energy penalty) or PO_NORM_ENERGY", i);
  return PO_OK;
}

std::atomic<int32_t> g_check_finite{0};

__global__ void k_zero_count(unsigned int* count) { *count = 0u; }

// Adds the number of non-finite entries of v[0, n) to *count (grid-stride; one atomic per block).
__global__ void __launch_bounds__(256) k_count_nonfinite(const double* __restrict__ v, int64_t n,
                                                         unsigned int* __restrict__ count) {
  __shared__ unsigned int part[256];
  unsigned int c = 0;
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256)
    c += std::isfinite(v[i]) ? 0u : 1u;
  part[threadIdx.x] = c;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0 && part[0] != 0u) atomicAdd(count, part[0]);
}

// With the check enabled: counts the non-finite entries of d_v[0, n) on the stream, waits for it,
// and returns PO_ERR_NUMERIC if there are any.
po_status check_finite(const double* d_v, int64_t n, const char* what, hipStream_t s) {
  if (!g_check_finite.load(std::memory_order_relaxed) || n <= 0) return PO_OK;
  Scratch cnt;
  PO_TRY(cnt.alloc(sizeof(unsigned int), s));
  unsigned int* d_c = static_cast<unsigned int*>(cnt.ptr);
  hipLaunchKernelGGL(k_zero_count, dim3(1), dim3(1), 0, s, d_c);
  PO_HIP(hipGetLastError());
  const int64_t blocks = std::min<int64_t>(1024, (n + 255) / 256);
  hipLaunchKernelGGL(k_count_nonfinite, dim3(unsigned(blocks)), dim3(256), 0, s, d_v, n, d_c);
  PO_HIP(hipGetLastError());
  unsigned int h_c = 0;
  PO_HIP(hipMemcpyAsync(&h_c, d_c, sizeof(h_c), hipMemcpyDeviceToHost, s));
  PO_HIP(hipStreamSynchronize(s));
  if (h_c != 0u) return set_error(PO_ERR_NUMERIC, "%u non-finite values in %s", h_c, what);
  return PO_OK;
}

// The evolution's checked output: J, or f when J is not requested.
po_status check_outputs(const Batch& b, const double* d_f, const double* d_J, hipStream_t s) {
  return d_J ? check_finite(d_J, b.n_pulses, "d_J", s) : check_finite(d_f, b.total_modes, "d_f", s);
}

}  // namespace

bool timer_start(hipStream_t s, hipEvent_t* e0) {
  {
    std::lock_guard<std::mutex> lk(g_timer_mu);
    if (!g_timer_on) return false;
  }
  if (hipEventCreate(e0) != hipSuccess) return false;
  if (hipEventRecord(*e0, s) != hipSuccess) {
    (void)hipEventDestroy(*e0);
    return false;
  }
  return true;
}

po_status timer_count(int n_pulses, const PulseDev* d_desc, const double* d_ranges, hipStream_t s) {
  unsigned long long* c;
  {
    std::lock_guard<std::mutex> lk(g_timer_mu);
    if (!g_timer_on || !g_counts) return PO_OK;
    c = g_counts;
  }
  return launch_count_mode_steps(n_pulses, d_desc, d_ranges, c, s);
}

void timer_stop(hipStream_t s, hipEvent_t e0) {
  hipEvent_t e1 = nullptr;
  if (hipEventCreate(&e1) != hipSuccess || hipEventRecord(e1, s) != hipSuccess) {
    (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    return;
  }
  std::lock_guard<std::mutex> lk(g_timer_mu);
  g_timer_events.emplace_back(e0, e1);
}

// ---------------------------------------------------------------------------------------------
// Allocation-free evaluation: every scratch buffer of po_evaluate_noalloc lives in this file-scope
// device array (each device holds its own copy until the process ends).  In host code `scratch`
// is only a stand-in for the symbol: its device address comes from hipGetSymbolAddress, taken once
// per device with that device current, and only that address is handed to kernels and copies.
// ---------------------------------------------------------------------------------------------
constexpr int kNoAllocMaxPulses = 4096;
constexpr size_t kNoAllocLimitBytes = size_t(64) << 20;
// Beyond the limit's own sizes: 32 bytes per line (at most 2^21 lines within the limit), up to 18 records
// more per pulse and what a descriptor exceeds 208 bytes by.
constexpr size_t kNoAllocScratchBytes = 2 * kNoAllocLimitBytes + kNoAllocMaxPulses * (18 * 8 * kSpecRec + sizeof(PulseDev) - 208) + 4096;
constexpr int kNoAllocMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

std::mutex g_noalloc_mu;                               // guards the two arrays below
void* g_scratch_dev[kNoAllocMaxDevices] = {};          // device address of `scratch`, per device
PulseDev g_noalloc_desc[kNoAllocMaxPulses];            // host staging of the pulse descriptors

// Device address of `scratch` on the current device (looked up on the first call there).
po_status noalloc_scratch(void** out) {
  int dev = -1;
  PO_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kNoAllocMaxDevices) return set_error(PO_ERR_UNSUPPORTED, "device %d out of range", dev);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return device_error(e == hipSuccess ? hipErrorInvalidSymbol : e, "hipGetSymbolAddress");
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return PO_OK;
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace po

using namespace po;

extern "C" {

int po_abi_version(void) { return 1; }

int32_t po_set_check_finite(int32_t enable) { return g_check_finite.exchange(enable ? 1 : 0); }

const char* po_last_error(void) { return g_error.c_str(); }

po_status po_pulse_synth(int32_t n, const po_pulse_spec* specs, const double* d_coeff, double* d_A, double* d_E,
                         double* d_A_edge, double* d_scale, void* stream) {
  if (n < 1) return set_error(PO_ERR_INVALID, "n_pulses must be >= 1");
  PO_TRY(check_specs(n, specs));
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, specs, nullptr, h.data(), &b));
  PO_TRY(check_device_range(d_coeff, sizeof(double) * b.total_coeff, 8, "d_coeff"));
  PO_TRY(check_device_range(d_A, sizeof(double) * 2 * b.total_rows, 8, "d_A"));
  if (d_E) PO_TRY(check_device_range(d_E, sizeof(double) * 2 * b.total_rows, 8, "d_E"));
  PO_TRY(check_device_range(d_A_edge, sizeof(double) * 4 * n, 8, "d_A_edge"));
  if (d_scale) PO_TRY(check_device_range(d_scale, sizeof(double) * n, 8, "d_scale"));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Work w;
  const DescWork dw(w, n);
  const SynthWork sw(w, n, b);
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  PO_TRY(synth_impl(w, sw, d_coeff, d_A, d_E, d_A_edge, d_scale, nullptr, s, b, d_desc));
  return check_finite(d_A, 2 * b.total_rows, "d_A", s);
}

po_status po_evolve_modes(int32_t n, const po_pulse_spec* specs, const po_grid* grids, const double* d_A,
                          const double* d_A_edge, double* d_f, double* d_J, const struct po_plan* plan, void* stream) {
  if (n < 1) return set_error(PO_ERR_INVALID, "n_pulses must be >= 1");
  PO_TRY(check_specs(n, specs));
  PO_TRY(check_grids(n, grids));
  if (!d_f && !d_J) return set_error(PO_ERR_INVALID, "at least one of d_f, d_J must be non-NULL");
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, specs, grids, h.data(), &b));
  PO_TRY(check_device_range(d_A, sizeof(double) * 2 * b.total_rows, 8, "d_A"));
  PO_TRY(check_device_range(d_A_edge, sizeof(double) * 4 * n, 8, "d_A_edge"));
  if (d_f) PO_TRY(check_device_range(d_f, sizeof(double) * b.total_modes, 8, "d_f"));
  if (d_J) PO_TRY(check_device_range(d_J, sizeof(double) * n, 8, "d_J"));
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (plan) {
    hipEvent_t e0 = nullptr;
    const bool timed = timer_start(s, &e0);
    PO_TRY(plan_evolve(plan, n, specs, grids, d_A, d_A_edge, d_f, d_J, s));
    if (timed) timer_stop(s, e0);
    return check_outputs(b, d_f, d_J, s);
  }
  Work w;
  const DescWork dw(w, n);
  const EvolveWork ew(w, b);
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  PO_TRY(evolve_impl(w, ew, b, d_desc, d_A, d_A_edge, false, d_f, d_J, s));
  return check_outputs(b, d_f, d_J, s);
}

po_status po_field_samples(int32_t n, const po_pulse_spec* specs, const double* d_coeff, int32_t n_sub,
                           const double* offsets, int32_t with_end, double* d_E, double* d_Ed, double* d_A,
                           double* d_A_edge, double* d_scale, void* stream) {
  if (n < 1) return set_error(PO_ERR_INVALID, "n_pulses must be >= 1");
  PO_TRY(check_specs(n, specs));
  if (n_sub < 1 || n_sub > kMaxSub) return set_error(PO_ERR_INVALID, "n_sub must be in [1, %d]", kMaxSub);
  if (!offsets) return set_error(PO_ERR_INVALID, "offsets is NULL");
  for (int r = 0; r < n_sub; ++r)
    if (!(offsets[r] >= 0.0 && offsets[r] <= 1.0)) return set_error(PO_ERR_INVALID, "offsets[%d] not in [0, 1]", r);
  if (!d_E && !d_Ed && !d_A && !d_A_edge)
    return set_error(PO_ERR_INVALID, "at least one of d_E, d_Ed, d_A, d_A_edge must be non-NULL");
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, specs, nullptr, h.data(), &b));
  int64_t rows = 0;
  for (int i = 0; i < n; ++i) {
    h[i].tab_off = rows;
    rows += int64_t(specs[i].nt) * n_sub + (with_end ? 1 : 0);
  }
  PO_TRY(check_device_range(d_coeff, sizeof(double) * b.total_coeff, 8, "d_coeff"));
  if (d_E) PO_TRY(check_device_range(d_E, sizeof(double) * 2 * rows, 8, "d_E"));
  if (d_Ed) PO_TRY(check_device_range(d_Ed, sizeof(double) * 2 * rows, 8, "d_Ed"));
  if (d_A) PO_TRY(check_device_range(d_A, sizeof(double) * 2 * rows, 8, "d_A"));
  if (d_A_edge) PO_TRY(check_device_range(d_A_edge, sizeof(double) * 4 * n, 8, "d_A_edge"));
  if (d_scale) PO_TRY(check_device_range(d_scale, sizeof(double) * n, 8, "d_scale"));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Work w;
  const DescWork dw(w, n);
  const SynthWork sw(w, n, b);
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  return launch_samples(b, d_desc, d_coeff, w.at<double>(sw.spec), w.at<double>(sw.part), w.at<double>(sw.scl), n_sub,
                        offsets, with_end ? 1 : 0, d_E, d_Ed, d_A, d_A_edge, d_scale, s);
}

po_status po_qke_modes(int32_t n, const po_pulse_spec* specs, const po_grid* grids, const double* d_E,
                       const double* d_Ed, const double* d_A, int32_t linear, double* d_f, double* d_J, void* stream) {
  if (n < 1) return set_error(PO_ERR_INVALID, "n_pulses must be >= 1");
  PO_TRY(check_specs(n, specs));
  PO_TRY(check_grids(n, grids));
  if (!d_f && !d_J) return set_error(PO_ERR_INVALID, "at least one of d_f, d_J must be non-NULL");
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, specs, grids, h.data(), &b));
  int64_t rows = 0;
  for (int i = 0; i < n; ++i) {
    h[i].tab_off = rows;
    rows += 2 * int64_t(specs[i].nt) + 1;
  }
  PO_TRY(check_device_range(d_E, sizeof(double) * 2 * rows, 8, "d_E"));
  PO_TRY(check_device_range(d_Ed, sizeof(double) * 2 * rows, 8, "d_Ed"));
  PO_TRY(check_device_range(d_A, sizeof(double) * 2 * rows, 8, "d_A"));
  if (d_f) PO_TRY(check_device_range(d_f, sizeof(double) * b.total_modes, 8, "d_f"));
  if (d_J) PO_TRY(check_device_range(d_J, sizeof(double) * n, 8, "d_J"));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Work w;
  const DescWork dw(w, n);
  const size_t o_units = w.add(sizeof(double) * size_t(b.total_units));
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  double* d_units = d_J ? w.at<double>(o_units) : nullptr;
  PO_TRY(launch_qke_grid(b, d_desc, d_E, d_Ed, d_A, linear ? 1 : 0, d_f, d_units, s));
  if (d_J) PO_TRY(launch_yield_from_units(b, d_desc, d_units, d_J, s));
  return PO_OK;
}

po_status po_evolve_modes_m4(int32_t n, const po_pulse_spec* specs, const po_grid* grids, const double* d_Ag,
                             const double* d_A_edge, double* d_f, double* d_J, void* stream) {
  if (n < 1) return set_error(PO_ERR_INVALID, "n_pulses must be >= 1");
  PO_TRY(check_specs(n, specs));
  PO_TRY(check_grids(n, grids));
  if (!d_f && !d_J) return set_error(PO_ERR_INVALID, "at least one of d_f, d_J must be non-NULL");
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, specs, grids, h.data(), &b));
  PO_TRY(check_device_range(d_Ag, sizeof(double) * 4 * b.total_rows, 16, "d_Ag"));
  PO_TRY(check_device_range(d_A_edge, sizeof(double) * 4 * n, 8, "d_A_edge"));
  if (d_f) PO_TRY(check_device_range(d_f, sizeof(double) * b.total_modes, 8, "d_f"));
  if (d_J) PO_TRY(check_device_range(d_J, sizeof(double) * n, 8, "d_J"));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Work w;
  const DescWork dw(w, n);
  const EvolveWork z(w, b);
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  double* d_units = d_J ? w.at<double>(z.units) : nullptr;
  PO_TRY(launch_evolve4(b, d_desc, d_Ag, d_A_edge, w.at<double>(z.ranges),
          z.split ? w.at<double>(z.prop) : nullptr, d_f, d_units, s));
  if (d_J) PO_TRY(launch_yield_from_units(b, d_desc, d_units, d_J, s));
  return PO_OK;
}

po_status po_evolve_modes_split(int32_t n, const po_pulse_spec* specs, const po_grid* grids, int32_t order,
                                const double* d_At, const double* d_A_edge, double* d_f, double* d_J, void* stream) {
  if (n < 1) return set_error(PO_ERR_INVALID, "n_pulses must be >= 1");
  if (order != 2 && order != 4) return set_error(PO_ERR_INVALID, "order must be 2 or 4");
  PO_TRY(check_specs(n, specs));
  PO_TRY(check_grids(n, grids));
  if (!d_f && !d_J) return set_error(PO_ERR_INVALID, "at least one of d_f, d_J must be non-NULL");
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, specs, grids, h.data(), &b));
  const int nsub = order == 2 ? 1 : 3;
  PO_TRY(check_device_range(d_At, sizeof(double) * 2 * nsub * b.total_rows, 16, "d_At"));
  PO_TRY(check_device_range(d_A_edge, sizeof(double) * 4 * n, 16, "d_A_edge"));
  if (d_f) PO_TRY(check_device_range(d_f, sizeof(double) * b.total_modes, 8, "d_f"));
  if (d_J) PO_TRY(check_device_range(d_J, sizeof(double) * n, 8, "d_J"));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Work w;
  const DescWork dw(w, n);
  const EvolveWork z(w, b);
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  double* d_units = d_J ? w.at<double>(z.units) : nullptr;
  PO_TRY(launch_evolve_split(b, order, d_desc, d_At, d_A_edge, w.at<double>(z.ranges),
          z.split ? w.at<double>(z.prop) : nullptr, d_f, d_units, s));
  if (d_J) PO_TRY(launch_yield_from_units(b, d_desc, d_units, d_J, s));
  return PO_OK;
}

po_status po_yield_gradient(int32_t n, const po_pulse_spec* specs, const po_grid* grids, const double* d_A,
                            const double* d_A_edge, double* d_J, double* d_gA, double* d_gedge, void* stream) {
  if (n < 1) return set_error(PO_ERR_INVALID, "n_pulses must be >= 1");
  PO_TRY(check_specs(n, specs));
  PO_TRY(check_grids(n, grids));
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, specs, grids, h.data(), &b));
  PO_TRY(check_device_range(d_A, sizeof(double) * 2 * b.total_rows, 8, "d_A"));
  PO_TRY(check_device_range(d_A_edge, sizeof(double) * 4 * n, 8, "d_A_edge"));
  PO_TRY(check_device_range(d_gA, sizeof(double) * 2 * b.total_rows, 8, "d_gA"));
  if (d_gedge) PO_TRY(check_device_range(d_gedge, sizeof(double) * 4 * n, 8, "d_gedge"));
  if (d_J) PO_TRY(check_device_range(d_J, sizeof(double) * n, 8, "d_J"));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Work w;
  const DescWork dw(w, n);
  const GradWork gw(w, h, b);
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  return yield_grad_impl(w, gw, b, d_desc, d_A, d_A_edge, false, d_J, d_gA, d_gedge, s);
}

po_status po_synth_gradient(int32_t n, const po_pulse_spec* specs, const double* d_coeff, const double* d_gA,
                            const double* d_gedge, double* d_grad, double* d_U, double* d_gU, void* stream) {
  if (n < 1) return set_error(PO_ERR_INVALID, "n_pulses must be >= 1");
  PO_TRY(check_specs(n, specs));
  PO_TRY(check_differentiable(n, specs));
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, specs, nullptr, h.data(), &b));
  PO_TRY(check_device_range(d_coeff, sizeof(double) * b.total_coeff, 8, "d_coeff"));
  PO_TRY(check_device_range(d_gA, sizeof(double) * 2 * b.total_rows, 8, "d_gA"));
  if (d_gedge) PO_TRY(check_device_range(d_gedge, sizeof(double) * 4 * n, 8, "d_gedge"));
  PO_TRY(check_device_range(d_grad, sizeof(double) * b.total_coeff, 8, "d_grad"));
  if (d_U) PO_TRY(check_device_range(d_U, sizeof(double) * n, 8, "d_U"));
  if (d_gU) PO_TRY(check_device_range(d_gU, sizeof(double) * b.total_coeff, 8, "d_gU"));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Work w;
  const DescWork dw(w, n);
  const SynthWork sw(w, n, b);
  const AdjointWork aw(w, n, b);
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  double *dA = w.at<double>(aw.A), *dE = w.at<double>(aw.E), *de = w.at<double>(aw.edge);
  double* dscale = w.at<double>(aw.scale);
  PO_TRY(synth_impl(w, sw, d_coeff, dA, dE, de, dscale, nullptr, s, b, d_desc));
  return launch_synth_adjoint(b, d_desc, d_coeff, d_gA, d_gedge, dA, de, dE, dscale, w.at<double>(aw.harm),
                              w.at<double>(aw.lines), d_grad,
                              d_U, d_gU, s);
}

po_status po_evaluate_gradient(int32_t n, const po_pulse_spec* specs, const po_grid* grids, const double* d_coeff,
                               double* d_J, double* d_grad, double* d_U, double* d_gU, void* stream) {
  if (n < 1) return set_error(PO_ERR_INVALID, "n_pulses must be >= 1");
  PO_TRY(check_specs(n, specs));
  PO_TRY(check_grids(n, grids));
  PO_TRY(check_differentiable(n, specs));
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, specs, grids, h.data(), &b));
  PO_TRY(check_device_range(d_coeff, sizeof(double) * b.total_coeff, 8, "d_coeff"));
  PO_TRY(check_device_range(d_J, sizeof(double) * n, 8, "d_J"));
  PO_TRY(check_device_range(d_grad, sizeof(double) * b.total_coeff, 8, "d_grad"));
  if (d_U) PO_TRY(check_device_range(d_U, sizeof(double) * n, 8, "d_U"));
  if (d_gU) PO_TRY(check_device_range(d_gU, sizeof(double) * b.total_coeff, 8, "d_gU"));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Work w;
  const DescWork dw(w, n);
  const SynthWork sw(w, n, b);
  const AdjointWork aw(w, n, b);
  const GradWork gw(w, h, b);
  const size_t o_gA = w.add(sizeof(double) * 2 * b.total_rows), o_ge = w.add(sizeof(double) * 4 * n);
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  double *dA = w.at<double>(aw.A), *dE = w.at<double>(aw.E), *de = w.at<double>(aw.edge);
  double *dscale = w.at<double>(aw.scale), *dgA = w.at<double>(o_gA), *dge = w.at<double>(o_ge);
  PO_TRY(synth_impl(w, sw, d_coeff, dA, dE, de, dscale, w.at<double>(gw.ranges), s, b, d_desc));
  PO_TRY(yield_grad_impl(w, gw, b, d_desc, dA, de, true, d_J, dgA, dge, s));
  return launch_synth_adjoint(b, d_desc, d_coeff, dgA, dge, dA, de, dE, dscale, w.at<double>(aw.harm),
                              w.at<double>(aw.lines), d_grad, d_U,
                              d_gU, s);
}

po_status po_pair_yield(int32_t n, const po_grid* grids, const double* d_f, double* d_J, void* stream) {
  if (n < 1) return set_error(PO_ERR_INVALID, "n_pulses must be >= 1");
  PO_TRY(check_grids(n, grids));
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, nullptr, grids, h.data(), &b));
  PO_TRY(check_device_range(d_f, sizeof(double) * b.total_modes, 8, "d_f"));
  PO_TRY(check_device_range(d_J, sizeof(double) * n, 8, "d_J"));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Work w;
  const DescWork dw(w, n);
  const size_t o_units = w.add(sizeof(double) * size_t(b.total_units));
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  PO_TRY(launch_unit_sums_from_f(b, d_desc, d_f, w.at<double>(o_units), s));
  PO_TRY(launch_yield_from_units(b, d_desc, w.at<double>(o_units), d_J, s));
  return check_finite(d_J, n, "d_J", s);
}

po_status po_evaluate(int32_t n, const po_pulse_spec* specs, const po_grid* grids, const double* d_coeff, double* d_A,
                      double* d_A_edge, double* d_scale, double* d_f, double* d_J, const struct po_plan* plan,
                      void* stream) {
  if (n < 1) return set_error(PO_ERR_INVALID, "n_pulses must be >= 1");
  PO_TRY(check_specs(n, specs));
  PO_TRY(check_grids(n, grids));
  if (!d_f && !d_J) return set_error(PO_ERR_INVALID, "at least one of d_f, d_J must be non-NULL");
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, specs, grids, h.data(), &b));
  PO_TRY(check_device_range(d_coeff, sizeof(double) * b.total_coeff, 8, "d_coeff"));
  PO_TRY(check_device_range(d_A, sizeof(double) * 2 * b.total_rows, 8, "d_A"));
  PO_TRY(check_device_range(d_A_edge, sizeof(double) * 4 * n, 8, "d_A_edge"));
  if (d_scale) PO_TRY(check_device_range(d_scale, sizeof(double) * n, 8, "d_scale"));
  if (d_f) PO_TRY(check_device_range(d_f, sizeof(double) * b.total_modes, 8, "d_f"));
  if (d_J) PO_TRY(check_device_range(d_J, sizeof(double) * n, 8, "d_J"));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Work w;
  const DescWork dw(w, n);
  const SynthWork sw(w, n, b);
  const EvolveWork ew(w, plan ? Batch{} : b);  // a plan has its own
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  PO_TRY(synth_impl(w, sw, d_coeff, d_A, nullptr, d_A_edge, d_scale, plan ? nullptr : w.at<double>(ew.ranges), s, b,
                    d_desc));
  PO_TRY(check_finite(d_A, 2 * b.total_rows, "d_A", s));
  if (plan) {
    hipEvent_t e0 = nullptr;
    const bool timed = timer_start(s, &e0);
    PO_TRY(plan_evolve(plan, n, specs, grids, d_A, d_A_edge, d_f, d_J, s));
    if (timed) timer_stop(s, e0);
    return check_outputs(b, d_f, d_J, s);
  }
  PO_TRY(evolve_impl(w, ew, b, d_desc, d_A, d_A_edge, true, d_f, d_J, s));
  return check_outputs(b, d_f, d_J, s);
}

po_status po_evaluate_noalloc(int32_t n, const po_pulse_spec* specs, const po_grid* grids, const double* d_coeff,
                              double* d_A, double* d_A_edge, double* d_scale, double* d_f, double* d_J, void* stream) {
  if (n < 1) return set_error(PO_ERR_INVALID, "n_pulses must be >= 1");
  if (n > kNoAllocMaxPulses) return set_error(PO_ERR_INVALID, "n_pulses must be <= %d", kNoAllocMaxPulses);
  PO_TRY(check_specs(n, specs));
  PO_TRY(check_grids(n, grids));
  if (!d_f && !d_J) return set_error(PO_ERR_INVALID, "at least one of d_f, d_J must be non-NULL");
  std::lock_guard<std::mutex> lk(g_noalloc_mu);
  Batch b;
  PO_TRY(build_batch(n, specs, grids, g_noalloc_desc, &b));
  const EvalSizes z = eval_sizes(n, b);
  // the documented limit: descriptors (208 bytes a pulse), 4 doubles a line, a partial per 256 nodes of the longest
  // normalised pulse, scales, unit sums and ranges; the array also has room for what is larger in it
  int64_t blocks = 1;
  for (int i = 0; i < n; ++i)
    if (specs[i].norm != PO_NORM_NONE) blocks = std::max<int64_t>(blocks, (int64_t(specs[i].nt) + 1 + 255) / 256);
  const size_t limit = align256(208 * size_t(n)) + align256(32 * size_t(b.total_lines)) +
                       align256(sizeof(double) * size_t(blocks) * size_t(n)) + align256(sizeof(double) * z.scl) +
                       align256(sizeof(double) * z.units) + align256(sizeof(double) * z.ranges);
  if (limit > kNoAllocLimitBytes)
    return set_error(PO_ERR_INVALID, "batch needs %zu bytes of scratch, the allocation-free path holds %zu", limit,
                     kNoAllocLimitBytes);
  const size_t o_desc = 0;
  const size_t o_spec = o_desc + align256(sizeof(PulseDev) * size_t(n));
  const size_t o_part = o_spec + align256(sizeof(double) * z.spec);
  const size_t o_scl = o_part + align256(sizeof(double) * z.part);
  const size_t o_units = o_scl + align256(sizeof(double) * z.scl);
  const size_t o_ranges = o_units + align256(sizeof(double) * z.units);
  const size_t need = o_ranges + align256(sizeof(double) * z.ranges);
  if (need > kNoAllocScratchBytes) return set_error(PO_ERR_INVALID, "batch needs %zu bytes of scratch", need);
  PO_TRY(check_device_range(d_coeff, sizeof(double) * b.total_coeff, 8, "d_coeff"));
  PO_TRY(check_device_range(d_A, sizeof(double) * 2 * b.total_rows, 8, "d_A"));
  PO_TRY(check_device_range(d_A_edge, sizeof(double) * 4 * n, 8, "d_A_edge"));
  if (d_scale) PO_TRY(check_device_range(d_scale, sizeof(double) * n, 8, "d_scale"));
  if (d_f) PO_TRY(check_device_range(d_f, sizeof(double) * b.total_modes, 8, "d_f"));
  if (d_J) PO_TRY(check_device_range(d_J, sizeof(double) * n, 8, "d_J"));
  void* base = nullptr;
  PO_TRY(noalloc_scratch(&base));
  unsigned char* sc = static_cast<unsigned char*>(base);
  hipStream_t s = static_cast<hipStream_t>(stream);
  PulseDev* d_desc = reinterpret_cast<PulseDev*>(sc + o_desc);
  PO_HIP(hipMemcpyAsync(d_desc, g_noalloc_desc, sizeof(PulseDev) * size_t(n), hipMemcpyHostToDevice, s));
  PO_TRY(launch_synth(b, d_desc, d_coeff, reinterpret_cast<double*>(sc + o_spec), reinterpret_cast<double*>(sc + o_part),
                      reinterpret_cast<double*>(sc + o_scl), d_A, nullptr, d_A_edge, d_scale,
                      reinterpret_cast<double*>(sc + o_ranges), s));
  // what the scratch array has left serves the time-split form of a small batch
  const size_t prop_bytes = sizeof(double) * kSlotDoubles * size_t(b.total_slots);
  double* d_prop = split_in_time(b) && prop_bytes <= kNoAllocScratchBytes - need ? reinterpret_cast<double*>(sc + need)
                                                                                  : nullptr;
  return evolve_into(b, d_desc, d_A, d_A_edge, d_f, d_J, s, reinterpret_cast<double*>(sc + o_units),
                     reinterpret_cast<double*>(sc + o_ranges), true, d_prop, false);
}

po_status po_timer_enable(int on) {
  std::lock_guard<std::mutex> lk(g_timer_mu);
  if (on && !g_counts) {
    void* p = nullptr;
    PO_HIP(hipMalloc(&p, sizeof(unsigned long long) * kSeriesVariants));
    PO_HIP(hipMemset(p, 0, sizeof(unsigned long long) * kSeriesVariants));
    g_counts = static_cast<unsigned long long*>(p);
  }
  g_timer_on = on != 0;
  return PO_OK;
}

po_status po_timer_mode_steps(uint64_t* counts, int32_t n) {
  if (!counts || n < 1) return set_error(PO_ERR_INVALID, "counts must hold at least one entry");
  unsigned long long h[kSeriesVariants] = {};
  {
    std::lock_guard<std::mutex> lk(g_timer_mu);
    if (g_counts) {
      PO_HIP(hipDeviceSynchronize());
      PO_HIP(hipMemcpy(h, g_counts, sizeof h, hipMemcpyDeviceToHost));
      PO_HIP(hipMemset(g_counts, 0, sizeof h));
    }
  }
  for (int i = 0; i < n; ++i) counts[i] = i < kSeriesVariants ? uint64_t(h[i]) : 0;
  return PO_OK;
}

po_status po_timer_read(double* ms_total, int64_t* calls) {
  std::vector<std::pair<hipEvent_t, hipEvent_t>> ev;
  {
    std::lock_guard<std::mutex> lk(g_timer_mu);
    ev.swap(g_timer_events);
  }
  double total = 0.0;
  po_status st = PO_OK;
  for (auto& p : ev) {
    float ms = 0.0f;
    hipError_t e = hipEventSynchronize(p.second);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, p.first, p.second);
    if (e != hipSuccess && st == PO_OK) st = device_error(e, "hipEventElapsedTime");
    total += ms;
    (void)hipEventDestroy(p.first);
    (void)hipEventDestroy(p.second);
  }
  if (ms_total) *ms_total = total;
  if (calls) *calls = int64_t(ev.size());
  return st;
}

static po_status check_de(const po_de_params* p) {
  if (!p) return set_error(PO_ERR_INVALID, "params is NULL");
  if (p->pop < 4) return set_error(PO_ERR_INVALID, "pop must be >= 4");
  if (p->dim < 1) return set_error(PO_ERR_INVALID, "dim must be >= 1");
  if (p->n_s < 0) return set_error(PO_ERR_INVALID, "n_s must be >= 0");
  if (!(p->F >= 0.0 && p->F <= 2.0)) return set_error(PO_ERR_INVALID, "F must be in [0, 2]");
  if (!(p->CR >= 0.0 && p->CR <= 1.0)) return set_error(PO_ERR_INVALID, "CR must be in [0, 1]");
  if (!(p->lo < p->hi) || !std::isfinite(p->lo) || !std::isfinite(p->hi))
    return set_error(PO_ERR_INVALID, "need finite lo < hi");
  return PO_OK;
}

po_status po_de_propose(const po_de_params* prm, int64_t generation, const double* d_pop, double* d_trial,
                        int32_t* d_idx, void* stream) {
  PO_TRY(check_de(prm));
  const size_t nd = size_t(prm->pop) * prm->dim;
  PO_TRY(check_device_range(d_pop, sizeof(double) * nd, 8, "d_pop"));
  PO_TRY(check_device_range(d_trial, sizeof(double) * nd, 8, "d_trial"));
  if (d_idx) PO_TRY(check_device_range(d_idx, sizeof(int32_t) * 4 * prm->pop, 4, "d_idx"));
  return launch_de_propose(*prm, generation, d_pop, d_trial, d_idx, static_cast<hipStream_t>(stream));
}

po_status po_de_select(const po_de_params* prm, double* d_pop, double* d_fit, const double* d_trial,
                       const double* d_trial_fit, const uint8_t* d_mask, void* stream) {
  PO_TRY(check_de(prm));
  const size_t nd = size_t(prm->pop) * prm->dim;
  PO_TRY(check_device_range(d_pop, sizeof(double) * nd, 8, "d_pop"));
  PO_TRY(check_device_range(d_fit, sizeof(double) * prm->pop, 8, "d_fit"));
  PO_TRY(check_device_range(d_trial, sizeof(double) * nd, 8, "d_trial"));
  PO_TRY(check_device_range(d_trial_fit, sizeof(double) * prm->pop, 8, "d_trial_fit"));
  if (d_mask) PO_TRY(check_device_range(d_mask, prm->pop, 1, "d_mask"));
  return launch_de_select(*prm, d_pop, d_fit, d_trial, d_trial_fit, d_mask, static_cast<hipStream_t>(stream));
}

po_status po_de_generation(const po_de_params* prm, int64_t generation, const po_pulse_spec* spec, const po_grid* grid,
                           double* d_pop, double* d_fit, double* d_trial, double* d_trial_fit, void* stream) {
  PO_TRY(check_de(prm));
  PO_TRY(check_specs(1, spec));
  PO_TRY(check_grids(1, grid));
  if (prm->dim != 4 * spec->n_s) return set_error(PO_ERR_INVALID, "dim must equal 4 n_s");
  const int32_t n = prm->pop;
  const size_t nd = size_t(n) * prm->dim;
  PO_TRY(check_device_range(d_pop, sizeof(double) * nd, 8, "d_pop"));
  PO_TRY(check_device_range(d_fit, sizeof(double) * n, 8, "d_fit"));
  PO_TRY(check_device_range(d_trial, sizeof(double) * nd, 8, "d_trial"));
  PO_TRY(check_device_range(d_trial_fit, sizeof(double) * n, 8, "d_trial_fit"));
  std::vector<po_pulse_spec> specs(n, *spec);
  std::vector<po_grid> grids(n, *grid);
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, specs.data(), grids.data(), h.data(), &b));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Work w;
  const DescWork dw(w, n);
  const SynthWork sw(w, n, b);
  const EvolveWork ew(w, b);
  const size_t o_A = w.add(sizeof(double) * 2 * b.total_rows), o_edge = w.add(sizeof(double) * 4 * n);
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  double *d_A = w.at<double>(o_A), *d_edge = w.at<double>(o_edge);
  PO_TRY(launch_de_propose(*prm, generation, d_pop, d_trial, nullptr, s));
  PO_TRY(synth_impl(w, sw, d_trial, d_A, nullptr, d_edge, nullptr, w.at<double>(ew.ranges), s, b, d_desc));
  PO_TRY(evolve_impl(w, ew, b, d_desc, d_A, d_edge, true, nullptr, d_trial_fit, s));
  PO_TRY(launch_de_select(*prm, d_pop, d_fit, d_trial, d_trial_fit, nullptr, s));
  return check_finite(d_trial_fit, n, "d_trial_fit", s);
}

static po_status check_jde(const po_jde_params* p) {
  if (!p) return set_error(PO_ERR_INVALID, "params is NULL");
  if (p->islands < 1 || p->islands > 64) return set_error(PO_ERR_INVALID, "islands must be in [1, 64]");
  if (p->pop < 4 || p->pop % p->islands != 0 || p->pop / p->islands < 4)
    return set_error(PO_ERR_INVALID, "pop must be a multiple of islands with at least 4 members per island");
  if (p->dim < 1) return set_error(PO_ERR_INVALID, "dim must be >= 1");
  if (p->n_s < 0) return set_error(PO_ERR_INVALID, "n_s must be >= 0");
  if (!(p->tau1 >= 0.0 && p->tau1 <= 1.0) || !(p->tau2 >= 0.0 && p->tau2 <= 1.0))
    return set_error(PO_ERR_INVALID, "tau1 and tau2 must be in [0, 1]");
  if (!(p->F_lo >= 0.0 && p->F_lo <= p->F_hi && p->F_hi <= 2.0))
    return set_error(PO_ERR_INVALID, "need 0 <= F_lo <= F_hi <= 2");
  if (!(p->lo < p->hi) || !std::isfinite(p->lo) || !std::isfinite(p->hi))
    return set_error(PO_ERR_INVALID, "need finite lo < hi");
  return PO_OK;
}

static po_status check_jde_state(const po_jde_params* prm, const double* d_pop, const double* d_fit,
                                 const double* d_fcr) {
  const size_t nd = size_t(prm->pop) * prm->dim;
  PO_TRY(check_device_range(d_pop, sizeof(double) * nd, 8, "d_pop"));
  if (d_fit) PO_TRY(check_device_range(d_fit, sizeof(double) * prm->pop, 8, "d_fit"));
  PO_TRY(check_device_range(d_fcr, sizeof(double) * 2 * prm->pop, 8, "d_fcr"));
  return PO_OK;
}

po_status po_jde_propose(const po_jde_params* prm, int64_t generation, const double* d_pop, const double* d_fcr,
                         double* d_trial, double* d_trial_fcr, int32_t* d_idx, void* stream) {
  PO_TRY(check_jde(prm));
  PO_TRY(check_jde_state(prm, d_pop, nullptr, d_fcr));
  PO_TRY(check_jde_state(prm, d_trial, nullptr, d_trial_fcr));
  if (d_idx) PO_TRY(check_device_range(d_idx, sizeof(int32_t) * 4 * prm->pop, 4, "d_idx"));
  return launch_jde_propose(*prm, generation, d_pop, d_fcr, d_trial, d_trial_fcr, d_idx,
                            static_cast<hipStream_t>(stream));
}

po_status po_jde_select(const po_jde_params* prm, double* d_pop, double* d_fit, double* d_fcr, const double* d_trial,
                        const double* d_trial_fit, const double* d_trial_fcr, const uint8_t* d_mask, void* stream) {
  PO_TRY(check_jde(prm));
  PO_TRY(check_jde_state(prm, d_pop, d_fit, d_fcr));
  PO_TRY(check_jde_state(prm, d_trial, d_trial_fit, d_trial_fcr));
  if (d_mask) PO_TRY(check_device_range(d_mask, prm->pop, 1, "d_mask"));
  return launch_jde_select(*prm, d_pop, d_fit, d_fcr, d_trial, d_trial_fit, d_trial_fcr, d_mask,
                           static_cast<hipStream_t>(stream));
}

po_status po_island_migrate(const po_jde_params* prm, double* d_pop, double* d_fit, double* d_fcr, void* stream) {
  PO_TRY(check_jde(prm));
  if (prm->dim > 64) return set_error(PO_ERR_INVALID, "migration supports dim <= 64");
  PO_TRY(check_jde_state(prm, d_pop, d_fit, d_fcr));
  return launch_island_migrate(*prm, d_pop, d_fit, d_fcr, static_cast<hipStream_t>(stream));
}

po_status po_jde_generation(const po_jde_params* prm, int64_t generation, const po_pulse_spec* spec, const po_grid* grid,
                            double* d_pop, double* d_fit, double* d_fcr, double* d_trial, double* d_trial_fit,
                            double* d_trial_fcr, void* stream) {
  PO_TRY(check_jde(prm));
  PO_TRY(check_specs(1, spec));
  PO_TRY(check_grids(1, grid));
  if (prm->dim != 4 * spec->n_s) return set_error(PO_ERR_INVALID, "dim must equal 4 n_s");
  PO_TRY(check_jde_state(prm, d_pop, d_fit, d_fcr));
  PO_TRY(check_jde_state(prm, d_trial, d_trial_fit, d_trial_fcr));
  const int32_t n = prm->pop;
  std::vector<po_pulse_spec> specs(n, *spec);
  std::vector<po_grid> grids(n, *grid);
  std::vector<PulseDev> h(n);
  Batch b;
  PO_TRY(build_batch(n, specs.data(), grids.data(), h.data(), &b));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Work w;
  const DescWork dw(w, n);
  const SynthWork sw(w, n, b);
  const EvolveWork ew(w, b);
  const size_t o_A = w.add(sizeof(double) * 2 * b.total_rows), o_edge = w.add(sizeof(double) * 4 * n);
  PO_TRY(w.alloc(s));
  PulseDev* d_desc = w.at<PulseDev>(dw.desc);
  PO_TRY(put_desc(h, d_desc, s));
  double *d_A = w.at<double>(o_A), *d_edge = w.at<double>(o_edge);
  PO_TRY(launch_jde_propose(*prm, generation, d_pop, d_fcr, d_trial, d_trial_fcr, nullptr, s));
  PO_TRY(synth_impl(w, sw, d_trial, d_A, nullptr, d_edge, nullptr, w.at<double>(ew.ranges), s, b, d_desc));
  PO_TRY(evolve_impl(w, ew, b, d_desc, d_A, d_edge, true, nullptr, d_trial_fit, s));
  return launch_jde_select(*prm, d_pop, d_fit, d_fcr, d_trial, d_trial_fit, d_trial_fcr, nullptr, s);
}

}  // extern "C"
