// C ABI of the MI355X-native FR right-hand side (declared in include/frmi.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/frmi.h"
#include "filter.hpp"
#include "filter_tet.hpp"
#include "hex.hpp"
#include "mlp.hpp"
#include "pyr.hpp"
#include "setup.hpp"
#include "tet.hpp"

using namespace frmi;

namespace {

thread_local std::string g_thread_err;

// x rounded to FP32, then split into bf16 hi = rne(x) and lo = rne(x - hi) (bit patterns).
uint16_t bf16_rne(float f) {
  uint32_t b;
  std::memcpy(&b, &f, 4);
  b += 0x7FFFu + ((b >> 16) & 1u);
  return (uint16_t)(b >> 16);
}
void bf16_split_host(double x, uint16_t& hi, uint16_t& lo) {
  const float xf = (float)x;
  hi = bf16_rne(xf);
  const uint32_t hb = (uint32_t)hi << 16;
  float hf;
  std::memcpy(&hf, &hb, 4);
  lo = bf16_rne(xf - hf);
}

struct DevBlock {
  int etype = 0;
  int64_t n = 0, E = 0;
  int nsp = 0, nfp = 0, nfaces = 0;
  int64_t canon_off = 0, native_off = 0;
  double* geo = nullptr;    // FP64 geometry
  void* geo_t = nullptr;    // geometry in the kernels' arithmetic type (== geo for FP64)
  int32_t* nbr_elem = nullptr;
  int32_t* nbr_info = nullptr;
  void* uf = nullptr;       // [nfp][5][E] traces of u (not tetrahedra)
  void* grad = nullptr;     // gradient [nsp][15][E]; hexahedra, and where common fluxes are formed once per
                            // pair: the points' viscous flux, [nsp][9][E], 12 values by tile
  void* gradf = nullptr;    // hexahedra: f_v.n, [nfp][4][E]; two-sided pyramids: gradient traces [nfp][15][E]
  void* fc = nullptr;       // [nfp][5][E] common fluxes, where they are stored
  void* cmet = nullptr;     // curved hexahedra: stored metric terms in the kernels' type (else NULL)
  int64_t elem_off = 0;     // offset of the block in the element numbering (both orders)
  int32_t* cpos = nullptr;  // native index -> canonical index within the block [E] (-1: padding)
  double* sown = nullptr;   // entropy filter: own min entropy [E]
  double* smin = nullptr;   // entropy filter: neighbourhood min entropy [E]
  int32_t* f_det = nullptr;   // entropy filter: slot + 1 of the last call that listed the element [n]
  int32_t* f_list = nullptr;  // candidates of the search, native ids [n]
  int32_t* f_cnt = nullptr;   // candidate counts, one slot per filter call since the last s_min pass
};

struct RefVec {
  double v[5] = {0, 0, 0, 0, 0};
};

}  // namespace

struct fr_ctx_s {
  fr_params prm;
  hipStream_t stream = nullptr;
  Setup host;
  std::vector<DevBlock> blocks;
  int32_t* perm = nullptr;
  int32_t* g_npos = nullptr;          // canonical -> native element index, all blocks [n_elem_total]
  std::vector<int32_t> h_cpos;        // native -> canonical element index, all blocks (host)
  int64_t canon_len = 0, native_len = 0;
  // RK workspace: stage state and the increment of one stage in the native dtype; FP64 form: the
  // accumulator (the embedded pair's first increment) and that pair's second and third; FP32
  // form: the increments of stages 1..3 block by block (see rk_inc, rk_accum)
  void* rk_stage = nullptr;
  double* rk_acc = nullptr;
  void* rk_k = nullptr;
  void* rk_kk = nullptr;
  int* flag = nullptr;
  std::string err;
  // entropy filter / MLP workspace (canonical element order)
  int64_t n_elem_total = 0;
  int f_slot = -1;              // candidate counter of the current filter call (compute_smin starts over)
  int32_t* f_k = nullptr;
  int32_t* f_evals = nullptr;
  int32_t* f_flag = nullptr;
  float* f_feat = nullptr;
  float* f_khat = nullptr;
  double* f_copy = nullptr;     // FP64 native state copy (training targets)
  float* m_w = nullptr;         // MLP parameters, Adam moments, input scaling
  float* m_m = nullptr;
  float* m_v = nullptr;
  float* m_scale = nullptr;
  float* m_loss = nullptr;
  float* m_scratch = nullptr;
  float* m_sqerr = nullptr;
  int32_t* m_idx = nullptr;
  int m_batch_cap = 0;
  bool mlp_ready = false;
  float* static_scratch = nullptr;  // this device's copy of the library's fixed scratch array
  // tetrahedral operators on the device (arithmetic type of the context)
  void* tet_opT = nullptr;    // [TET_KP][TET_MP] transposed divergence operator
  void* tet_ogT = nullptr;    // [TGS_K][TGR_M] transposed stacked gradient operator, face-sparse row order
  void* tet_opH = nullptr;    // BF16x3 split of the divergence operator: hi [TET_MP][TET_KP16], then lo
  void* tet_ogH = nullptr;    // BF16x3 split of the gradient operator: hi [TGR_M][TGR_K], then lo
  double* rk_x0 = nullptr;    // adaptive stepping in the FP32 form: u_n
  double* rk_part = nullptr;   // adaptive stepping: per-workgroup partial sums of the norm
  double* rk_s64 = nullptr;   // FP64 stage state of the filtered FP32 form
  int32_t* tet_src = nullptr;
  void* pyr_ops = nullptr;    // pyramids: It [55][85], Dt [3][55][55], Lt [85][55] in the context's type
  double* tet_ftab = nullptr; // entropy filter on tetrahedra: modal operators, weights, multiplicities
  // training-data collection during filtered RK steps (fr_mlp_collect)
  bool collecting = false;
  float* col_x = nullptr;
  int32_t* col_k = nullptr;
  int64_t col_cap = 0, col_n = 0, col_seen = 0;
  // per-kernel event timing
  bool prof = false;
  struct ProfEv { int id; hipEvent_t a, b; };
  std::vector<std::string> prof_names;
  std::vector<ProfEv> prof_events;
  int prof_begin(const char* name) {
    if (!prof) return -1;
    int id = -1;
    for (size_t i = 0; i < prof_names.size(); ++i) if (prof_names[i] == name) id = (int)i;
    if (id < 0) { id = (int)prof_names.size(); prof_names.push_back(name); }
    ProfEv ev{id, nullptr, nullptr};
    if (hipEventCreate(&ev.a) != hipSuccess || hipEventCreate(&ev.b) != hipSuccess) return -1;
    (void)hipEventRecord(ev.a, stream);
    prof_events.push_back(ev);
    return (int)prof_events.size() - 1;
  }
  void prof_end(int k) {
    if (k >= 0) (void)hipEventRecord(prof_events[k].b, stream);
  }
  void prof_clear() {
    for (auto& e : prof_events) { (void)hipEventDestroy(e.a); (void)hipEventDestroy(e.b); }
    prof_events.clear();
    prof_names.clear();
  }
};

// Fixed device scratch of fr_mlp_grad_static: per-sample quantities (MLP_SS floats each)
// of up to FR_MLP_STATIC_MAX_BATCH samples, then their squared errors.  Each GPU holds its
// own copy; host code uses only the device address taken once per device at setup.
constexpr int64_t kStaticScratchFloats = (int64_t)FR_MLP_STATIC_MAX_BATCH * (MLP_SS + 1);
static __device__ __align__(256) float scratch[kStaticScratchFloats];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_addr[kMaxDevices] = {};
bool g_scratch_done[kMaxDevices] = {};

// The current device's address of `scratch` (looked up once per device), or nullptr.
float* static_scratch_address() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_done[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
      (void)hipGetLastError();
      ptr = nullptr;
    }
    g_scratch_addr[dev] = (float*)ptr;
    g_scratch_done[dev] = true;
  }
  return g_scratch_addr[dev];
}

}  // namespace

namespace {

fr_status fail(fr_ctx c, fr_status s, const std::string& msg) {
  if (c) c->err = msg;
  else g_thread_err = msg;
  return s;
}

#define HIP_TRY(ctx, call)                                                                  \
  do {                                                                                      \
    hipError_t e_ = (call);                                                                 \
    if (e_ != hipSuccess) return fail(ctx, FR_ERR_DEVICE, std::string(#call ": ") + hipGetErrorString(e_)); \
  } while (0)

template <typename T>
fr_status dalloc(fr_ctx c, T** p, size_t count) {
  *p = nullptr;
  if (count == 0) count = 1;
  hipError_t e = hipMalloc((void**)p, count * sizeof(T));
  if (e != hipSuccess) return fail(c, FR_ERR_ALLOC, std::string("hipMalloc: ") + hipGetErrorString(e));
  return FR_OK;
}

Phys phys_of(const fr_params& p) {
  Phys ph;
  ph.gamma = p.gamma;
  ph.mu = p.mu;
  ph.prandtl = p.prandtl;
  ph.beta = p.ldg_beta;
  ph.tau = p.ldg_tau;
  ph.riemann = p.riemann;
  return ph;
}

// ------------------------------------------------------------ layout kernels
// Canonical [elem][var][pt] (input element order) <-> native [pt][var][E] (native
// element order, cpos: native -> canonical element, -1 for padding).  A transpose: a block
// takes 32 native elements and up to 8 (or 40) points through LDS, so that native rows move in
// 32-element segments and canonical rows in segments of whole chunks (element by element,
// in any element order), where a grid-stride loop over one side touches a cache line per
// lane on the other.  Bound by HBM; the loads of a thread go out in rounds of eight before any is
// used (one at a time, packing a small mesh waited for five latencies in turn).  Rows of 33 values:
// the transposed accesses fall on different banks.  fr_unpack64 of 196,608 tetrahedra, renumbered
// (550 MB moved): 666 -> 125 us (4.4 TB/s), fr_pack64 680 -> 146; of 32,768 p = 3 hexahedra (168 MB):
// 107 -> 26 us (6.4 TB/s), packing 57 -> 29.
constexpr int LT_E = 32, LT_NT = 256;
template <int NSP, int MAXPC>
struct LayoutCfg {
  static constexpr int NCH = (NSP + MAXPC - 1) / MAXPC, PC = (NSP + NCH - 1) / NCH;
};

// T: the native type; in the FP32 deviation form ref is subtracted on the way in and added
// on the way out (zero for a right-hand side; unused in FP64).
template <typename T, int NSP, int MAXPC, bool PACK>
__global__ void __launch_bounds__(LT_NT) k_layout(const double* __restrict__ canon_in, double* __restrict__ canon_out,
                                                  const T* __restrict__ nat_in, T* __restrict__ nat_out,
                                                  const int32_t* __restrict__ cpos, int64_t E, RefVec ref) {
  constexpr int PC = LayoutCfg<NSP, MAXPC>::PC, NCH = LayoutCfg<NSP, MAXPC>::NCH, NR = 5 * PC, LD = LT_E + 1;
  __shared__ T tile[NR * LD];                    // [v][point of the chunk][el]
  __shared__ int32_t cp[LT_E];
  const int64_t blk = xcd_block();
  const int64_t e0 = blk / NCH * LT_E;
  const int p0 = (int)(blk % NCH) * PC, np = min(PC, NSP - p0);
  const int t = threadIdx.x;
  if (t < LT_E) cp[t] = cpos[e0 + t];
  const int el = t % LT_E, r0 = t / LT_E;
  // every load of a thread is issued before the first is used (a mesh of one tile waits for
  // one memory latency, not for one per row)
  constexpr int NI = (NR + LT_NT / LT_E - 1) / (LT_NT / LT_E);
  if constexpr (!PACK) {
    T x[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = min(r0 + i * (LT_NT / LT_E), 5 * np - 1);
      x[i] = nat_in[((int64_t)p0 * 5 + r) * E + e0 + el];
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = r0 + i * (LT_NT / LT_E);
      if (r < 5 * np) tile[((r % 5) * PC + r / 5) * LD + el] = x[i];
    }
  }
  __syncthreads();
  // value q of the chunk: canonical element, point, variable (pt fastest, as in memory)
  constexpr int NQ = (LT_E * NR + LT_NT - 1) / LT_NT, RD = NQ < 8 ? NQ : 8;
#pragma unroll
  for (int i0 = 0; i0 < NQ; i0 += RD) {
    double x[PACK ? RD : 1];
    if constexpr (PACK) {
#pragma unroll
      for (int i = 0; i < RD; ++i) {
        const int q = t + (i0 + i) * LT_NT, pt = q % PC, ev = q / PC;
        const bool ok = q < LT_E * NR && pt < np;
        const int ce = ok ? cp[ev / 5] : -1;
        x[i] = canon_in[ce >= 0 ? ((int64_t)ce * 5 + ev % 5) * NSP + p0 + pt : 0];
      }
    }
#pragma unroll
    for (int i = 0; i < RD; ++i) {
      const int q = t + (i0 + i) * LT_NT, pt = q % PC, ev = q / PC, v = ev % 5;
      if (q >= LT_E * NR || pt >= np) continue;
      const int ce = cp[ev / 5];
      T* w = &tile[(v * PC + pt) * LD + ev / 5];
      if constexpr (PACK)
        *w = ce >= 0 ? (T)(x[i] - ref.v[v]) : (T)(sizeof(T) == 8 && (v == 0 || v == 4) ? 1 : 0);
      else if (ce >= 0)
        canon_out[((int64_t)ce * 5 + v) * NSP + p0 + pt] = sizeof(T) == 8 ? (double)*w : (double)*w + ref.v[v];
    }
  }
  if constexpr (PACK) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = r0 + i * (LT_NT / LT_E);
      if (r < 5 * np) nat_out[((int64_t)p0 * 5 + r) * E + e0 + el] = tile[((r % 5) * PC + r / 5) * LD + el];
    }
  }
}

// The same for few values: a thread per value of the native rows, no staging (its cache lines on
// the canonical side are touched by many threads, which costs nothing while they fit L2).
template <typename T, bool PACK>
__global__ void __launch_bounds__(256) k_layout_few(const double* __restrict__ canon_in, double* __restrict__ canon_out,
                                                    const T* __restrict__ nat_in, T* __restrict__ nat_out,
                                                    const int32_t* __restrict__ cpos, int64_t E, int nsp, RefVec ref) {
  const int64_t e = (int64_t)blockIdx.x * 64 + threadIdx.x;
  const int row = blockIdx.y * 4 + threadIdx.y, v = row % 5, pt = row / 5;
  if (pt >= nsp) return;
  const int64_t i = (int64_t)row * E + e;
  const int ce = cpos[e];
  const int64_t c = ((int64_t)ce * 5 + v) * nsp + pt;
  if constexpr (PACK) {
    nat_out[i] = ce >= 0 ? (T)(canon_in[c] - ref.v[v]) : (T)(sizeof(T) == 8 && (v == 0 || v == 4) ? 1 : 0);
  } else {
    const T x = nat_in[i];
    if (ce >= 0) canon_out[c] = sizeof(T) == 8 ? (double)x : (double)x + ref.v[v];
  }
}

template <typename T, bool PACK>
fr_status layout_block(fr_ctx c, const DevBlock& b, const double* cin, double* cout, const T* nin, T* nout, RefVec ref) {
  if (b.E % 64 != 0) return fail(c, FR_ERR_STATE, "block not padded to 64 elements");
  const int64_t tiles = b.E / LT_E, values = b.E * 5 * b.nsp;
  // kernel times, us, pack / unpack.  Few values, by a thread each / by tiles: 64 p = 2 hexahedra 2.2 / 4.1
  // and 2.3 / 3.6; 6,144 p = 1 3.3 / 3.9 and 3.4 / 3.3 (245,760 values); 2,048 p = 2 3.6 / 4.3 and 3.6 / 4.0;
  // 4,096 p = 2 4.8 / 4.5 and 5.3 / 4.4 (552,960); 1,024 p = 4 5.7 / 4.7 and 5.8 / 4.4
  if (values <= 262144) {
    const dim3 grid((unsigned)(b.E / 64), (unsigned)((5 * b.nsp + 3) / 4));
    k_layout_few<T, PACK><<<grid, dim3(64, 4), 0, c->stream>>>(cin, cout, nin, nout, b.cpos, b.E, b.nsp, ref);
    return FR_OK;
  }
  // chunks of 8 points (more, smaller blocks) or 40: 4,096 p = 4 hexahedra 9.7 / 12.1 and 9.2 / 9.7;
  // 32,768 p = 3 29.1 / 33.5 and 26.1 / 28.9 (10.5 M values).  Unpacking takes the larger ones past 16 M
  // values, when both sides no longer fit the 256 MB last-level cache (32,768 p = 4 81 / 97 and 79.5 / 64.8;
  // 196,608 tetrahedra 146 / 154 and 148 / 125), and past 3 M where one of them holds all points, so that an
  // element's canonical values leave in one piece: 24,480 tetrahedra after a right-hand side 15.2 / 13.1,
  // 18,432 12.0 / 10.7, 12,416 (2.2 M values) 8.7 / 9.4; 32,768 p = 2 14.3 / 12.9
  const bool large = !PACK && values >= (int64_t)(b.nsp <= 40 ? 3 : 16) << 20;
#define FR_LAYOUT(NSP)                                                                                          \
  case NSP:                                                                                                     \
    if (!large)                                                                                                 \
      k_layout<T, NSP, 8, PACK><<<(unsigned)(tiles * LayoutCfg<NSP, 8>::NCH), LT_NT, 0, c->stream>>>(            \
          cin, cout, nin, nout, b.cpos, b.E, ref);                                                              \
    else if constexpr (!PACK)                                                                                   \
      k_layout<T, NSP, 40, PACK><<<(unsigned)(tiles * LayoutCfg<NSP, 40>::NCH), LT_NT, 0, c->stream>>>(          \
          cin, cout, nin, nout, b.cpos, b.E, ref);                                                              \
    break
  switch (b.nsp) {
    FR_LAYOUT(8);
    FR_LAYOUT(27);
    FR_LAYOUT(64);
    FR_LAYOUT(125);
    FR_LAYOUT(35);
    FR_LAYOUT(55);
    default: return fail(c, FR_ERR_UNSUPPORTED, "points per element");
  }
#undef FR_LAYOUT
  return FR_OK;
}

// Per-element values from native to canonical element order (both global numberings).
__global__ void k_elem_to_canon(const int32_t* __restrict__ src, const int32_t* __restrict__ npos, int64_t n,
                                int32_t* __restrict__ dst) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = src[npos[i]];
}

// ------------------------------------------------------------ RK4 kernels
// stage 1: acc = u + dt/6 k ; st = u + dt/2 k  (FP64 state; increments FP64 or FP32)
template <typename KT>
__global__ void k_rk_first(const double* __restrict__ u, const KT* __restrict__ k, double* __restrict__ acc,
                           double* __restrict__ st, int64_t n, double b, double c) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const double ui = u[i], ki = (double)k[i];
    acc[i] = ui + b * ki;
    st[i] = ui + c * ki;
  }
}
// middle stages: acc += b k ; st = u + c k
template <typename KT>
__global__ void k_rk_mid(const double* __restrict__ u, const KT* __restrict__ k, double* __restrict__ acc,
                         double* __restrict__ st, int64_t n, double b, double c) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const double ki = (double)k[i];
    acc[i] += b * ki;
    st[i] = u[i] + c * ki;
  }
}
// last: u = acc + b k
template <typename KT>
__global__ void k_rk_last(double* __restrict__ u, const KT* __restrict__ k, const double* __restrict__ acc,
                          int64_t n, double b) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    u[i] = acc[i] + b * (double)k[i];
}

// ------------------------------------------------------------ check kernel
__global__ void k_check(const double* __restrict__ u, int64_t n, int64_t E, int nsp, double gm1, int* flag) {
  const int64_t total = (int64_t)nsp * n;
  int bad = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t e = i % n;
    const int pt = (int)(i / n);
    double w[5];
    for (int v = 0; v < 5; ++v) w[v] = u[((int64_t)pt * 5 + v) * E + e];
    const double p = gm1 * (w[4] - 0.5 * (w[1] * w[1] + w[2] * w[2] + w[3] * w[3]) / w[0]);
    bool ok = true;
    for (int v = 0; v < 5; ++v) ok = ok && isfinite(w[v]);
    ok = ok && w[0] > 0 && p > 0 && isfinite(p);
    bad |= !ok;
  }
  if (bad) atomicOr(flag, 1);
}

int grid_for(int64_t n, int threads) {
  int64_t g = (n + threads - 1) / threads;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (int)g;
}

// ------------------------------------------------------------ FP32-form kernels
// Deviation of the FP64 state from the reference state, rounded to FP32.
__global__ void k_to_dev(const double* __restrict__ u, float* __restrict__ w, int64_t n, int64_t E, RefVec ref) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    w[i] = (float)(u[i] - ref.v[(i / E) % 5]);
}
// ------------------------------------------------------------ embedded-pair stages
// The embedded pair with the increments kept: with x_i = u_n + dt sum_{j<i} b_j k_j,
//   Y = x_i + dt a_{i+1,i} k_i  (the next stage state; in the native dtype, FP32 deviation in
// the FP32 form).  x_i is summed again from the kept increments, in the registers' order, so
// that a stage reads and writes neither a running state nor an error register, and the last
// stage forms the new state, the saved u_n and the error norm in one pass.  Padding lanes take no
// increment (nothing writes theirs, and the buffers are shared with RK4's).  Bound by its bytes,
// per FP64 value and attempt 152 instead of 208 (FP32 form 100 instead of
// 180).  An attempt on 13,800 p = 3 Navier-Stokes hexahedra in FP64, right-hand sides included:
// 864 -> 769 us.
template <typename KT>
struct LsK {
  const KT* k[4];
  double xb[4], ed[4], ya;
};

template <typename KT, int I>
__global__ void __launch_bounds__(256) k_lsrk_stage(const double* __restrict__ X, LsK<KT> A, KT* __restrict__ Y,
                                                    int64_t E, int64_t n_real, int rows, RefVec ref) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= E) return;
  const bool real = e < n_real;
  for (int row = blockIdx.y; row < rows; row += gridDim.y) {
    const int64_t i = (int64_t)row * E + e;
    double x = X[i], k[I + 1];
#pragma unroll
    for (int j = 0; j <= I; ++j) k[j] = real ? (double)A.k[j][i] : 0.0;
#pragma unroll
    for (int j = 0; j < I; ++j) x = x + A.xb[j] * k[j];
    Y[i] = (KT)(x + A.ya * k[I] - (sizeof(KT) == 4 ? ref.v[row % 5] : 0.0));
  }
}

// The last stage: X = u_n + dt sum_j b_j k_j, X0 = u_n, and the sums of (err / scale)^2 of the
// real elements, err = dt sum_j (b_j - b^_j) k_j.
template <typename KT>
__global__ void __launch_bounds__(256) k_lsrk_last(double* __restrict__ X, LsK<KT> A, double* __restrict__ X0,
                                                   int64_t n, int64_t E, int64_t n_real, double atol, double rtol,
                                                   double* __restrict__ part) {
  __shared__ double red[256];
  double a = 0.0;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  const int64_t de = step % E;
  int64_t el = i0 % E;
  for (int64_t i = i0; i < n; i += step) {
    const double x0 = X[i];
    double k[4], x = x0, err = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) k[j] = el < n_real ? (double)A.k[j][i] : 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x = x + A.xb[j] * k[j];
      err = err + A.ed[j] * k[j];
    }
    X[i] = x;
    X0[i] = x0;
    if (el < n_real) {
      const double q = err / (atol + rtol * fmax(fabs(x0), fabs(x)));
      a += q * q;
    }
    el += de;
    if (el >= E) el -= E;
  }
  red[threadIdx.x] = a;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// RK stages of the FP32 form: FP64 state, FP32 increments kept per stage (k1, k2, k3; half the
// bytes of an FP64 accumulator read and written by every stage) and FP32 stage deviations.
// The last stage adds them in FP64 in the accumulator's order, so the sums are the same bits.
// HBM-bound: 84 bytes per value and step instead of 112.  Rows (blockIdx.y) of one variable,
// so a value's reference entry costs no division by E; two values per thread (E is a
// multiple of 64).  Padding lanes take no increment (nothing writes theirs).  32,768 p = 3
// hexahedra: 54.7 -> 39.8 us per stage on average.
struct Rk32 {
  double* u;                                      // u_n, and the new state (last stage)
  const float *k1, *k2, *k3, *k;
  float* st;
  double* s64;                                    // FP64 stage state as well, or null
  double b1, b2, c;
};
template <bool LAST>
__global__ void __launch_bounds__(256) k_rk32(Rk32 A, int64_t E, int64_t n_real, int rows, RefVec ref) {
  const int64_t e = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 2;
  if (e >= E) return;
  const bool r0 = e < n_real, r1 = e + 1 < n_real;
  auto inc = [&](const float* p, int64_t i) {
    const float2 x = *reinterpret_cast<const float2*>(p + i);
    return make_float2(r0 ? x.x : 0.0f, r1 ? x.y : 0.0f);
  };
  for (int row = blockIdx.y; row < rows; row += gridDim.y) {
    const int64_t i = (int64_t)row * E + e;
    const double rv = ref.v[row % 5];
    const double u0 = A.u[i], u1 = A.u[i + 1];    // the caller's array: 8-byte alignment
    const float2 k = inc(A.k, i);
    double s0, s1;
    if constexpr (LAST) {
      const float2 k1 = inc(A.k1, i);
      const float2 k2 = inc(A.k2, i);
      const float2 k3 = inc(A.k3, i);
      s0 = rk4_sum(u0, k1.x, k2.x, k3.x, k.x, A.b1, A.b2);
      s1 = rk4_sum(u1, k1.y, k2.y, k3.y, k.y, A.b1, A.b2);
      A.u[i] = s0;
      A.u[i + 1] = s1;
    } else {
      s0 = fma(A.c, (double)k.x, u0);
      s1 = fma(A.c, (double)k.y, u1);
      if (A.s64) {
        A.s64[i] = s0;
        A.s64[i + 1] = s1;
      }
    }
    *reinterpret_cast<float2*>(A.st + i) = make_float2((float)(s0 - rv), (float)(s1 - rv));
  }
}

// ------------------------------------------------------------ hex dispatch
template <int P>
struct HexCfg;
template <> struct HexCfg<1> { static constexpr int NE = 64; };
template <> struct HexCfg<2> { static constexpr int NE = 32; };
template <> struct HexCfg<3> { static constexpr int NE = 16; };
template <> struct HexCfg<4> { static constexpr int NE = 8; };
// element tile of the Euler divergence with the directions side by side (its LDS holds 15
// values per point and element)
template <typename T, int P>
struct DivEulCfg { static constexpr int NE = P == 1 ? 32 : (P == 2 ? 16 : (P == 3 || sizeof(T) == 4 ? 8 : 4)); };
// Most blocks for which the Euler divergence takes its directions side by side.  A whole
// right-hand side (with hex_trace where a form launches it) in turn / side by side, over meshes in
// order, of ragged sides and renumbered, straight and curved (the range over the three):
//   p = 3, p = 4 (all forms): 1.01-1.72 to 256 blocks (every block has a CU of its own),
//     0.50-1.13 from 288 on;
//   p = 1 FP64 straight: 1.54-1.93 to 256, 0.96-1.22 to 768, 0.73-0.96 from 896;
//   p = 2 FP32 straight: 1.63-1.78 to 256, 0.98-1.10 to 512, 0.63-0.92 from 640;
//   p = 1 FP32 straight: 1.17-1.57 to 768, 0.92-1.02 at 1,024, 0.72-0.90 from 1,536;
//   p = 2 FP64 straight: 1.02-1.38 to 768, 0.95-1.24 above (renumbered meshes lose);
//   p = 2 FP32 curved: 1.15-1.42 to 768, 0.94-1.18 above (renumbered meshes lose);
//   p = 1 curved: 1.00-2.15, p = 2 FP64 curved: 1.15-2.32, to 8,192 blocks, the largest timed.
constexpr int64_t kAnyBlocks = INT64_MAX;
template <typename T, int P, bool CUR>
constexpr int64_t wide_blocks() {
  if (CUR && (P == 1 || (P == 2 && sizeof(T) == 8))) return kAnyBlocks;
  if ((P == 1 && sizeof(T) == 4) || (P == 2 && (CUR || sizeof(T) == 8))) return 768;
  return 256;
}
// Element tile of the NS gradient and the threads per column of an element (its LDS holds 15
// values per point and element).  28^3 p = 4 FP64, us: 8 elements and 2 threads 223, 4 and 5
// 251, 8 and 3 436 (over the registers of its 10 waves); 32^3 p = 3 FP64: 2 threads 147, 4 173,
// 1 191; FP32 28^3 p = 4: 8 and 5 113, 8 and 2 141, 16 and 2 142; 32^3 p = 3: 16 elements and
// 2 threads 73, 4 threads 75, 8 and 4 78; 40^3 p = 2: 3 threads 76, 1 118.  Whole right-hand
// sides, us, here / half the elements / other threads: p = 1, 48^3 (1 thread) FP64 256 / 258 / 274,
// FP32 94 / 99 / 99, curved 254 / 251 / 258 and 110 / 109 / 109; curved p = 2, 36^3 (1) 287 / 294 / 395
// and 135 / 137 / 160; curved p = 3, 28^3 (4) 297 / 308 / 310 and 130 / 128 / 127; curved p = 4,
// 8,400 elements (FP64 3, FP32 2) 270 / 279 / 301 and 102 / 105 / 122.  Half the elements would gain in
// FP32 p = 3 straight (28^3 107 / 100) and 2-8 % on meshes of some hundred elements.
template <typename T, int P>
struct HexGradCfg {
  static constexpr int NE = P == 4 ? 8 : (sizeof(T) == 8 ? 1 : 2) * (P == 1 ? 32 : (P == 2 ? 16 : 8));
  static constexpr int KT = P == 1 ? 2 : (P == 2 ? 3 : (P == 3 || sizeof(T) == 8 ? 2 : 5));
};
// element tile of the NS divergence (its LDS holds 10 or 15 values per point and element)
template <typename T, int P>
struct DivNsCfg { static constexpr int NE = (sizeof(T) == 8 ? 8 : 16) / (P == 4 ? 2 : 1) * (P <= 2 ? 2 : 1); };

template <typename T>
HexK<T> hexk_of(const HexOps& H) {
  HexK<T> k;
  for (int a = 0; a < 5; ++a) {
    k.x[a] = (T)H.x[a]; k.lm[a] = (T)H.lm[a]; k.lp[a] = (T)H.lp[a];
    k.cp[a] = (T)H.cp[a]; k.cm[a] = (T)H.cm[a];
    for (int b = 0; b < 5; ++b) k.Dh[a][b] = (T)H.Dh[a][b];
  }
  return k;
}

template <typename T>
RefState<T> ref_of(const fr_params& p) {
  RefState<T> R;
  R.rho0 = (T)p.u_ref[0];
  R.E0 = (T)p.u_ref[4];
  R.p0 = (T)((p.gamma - 1.0) * p.u_ref[4]);
  R.H0 = (T)(p.u_ref[4] + (p.gamma - 1.0) * p.u_ref[4]);
  return R;
}

int side_mode_of(double beta) { return beta == 0.5 ? 1 : (beta == -0.5 ? -1 : 0); }

// Tetrahedra whose gradient kernel forms the common fluxes, once per pair: a one-sided switch
// (side_mode != 0), FP32 or straight elements (see tet_rhs).
constexpr bool tet_can_pair(bool f32, bool curved) { return f32 || !curved; }

template <typename T, bool DEV, int P, bool CUR>
fr_status hex_rhs_p(fr_ctx c, DevBlock& b, const T* u, T* r) {
  constexpr int N1 = P + 1, NE = HexCfg<P>::NE, NT = NE * N1 * N1;
  Conn C{b.nbr_elem, b.nbr_info, c->perm, c->host.perm_stride};
  const fr_params& p = c->prm;
  const HexK<T> K = hexk_of<T>(c->host.hex);
  const RefState<T> R = ref_of<T>(p);
  const T* geo = (const T*)b.geo_t;
  const T* cm = (const T*)b.cmet;
  T* uf = (T*)b.uf;
  T* grad = (T*)b.grad;
  T* gradf = (T*)b.gradf;
  const int sm = side_mode_of(p.ldg_beta);
  const int64_t trace_threads = b.E * 3 * N1 * N1;
  static const std::string sfx =
      std::string(CUR ? "_cur" : "") + (sizeof(T) == 8 ? "" : "_f32") + "_p" + std::to_string(P);
  constexpr int NEe = DivEulCfg<T, P>::NE;
  constexpr int64_t wide_most = wide_blocks<T, P, CUR>();
  const bool wide = p.system == FR_EULER && b.E / NEe <= wide_most;
  int pk = 0;
  if (!wide || !wide_own_traces<T, P, CUR>()) {
    pk = c->prof_begin(("hex_trace" + sfx).c_str());
    hex_trace<T, P><<<(unsigned)((trace_threads + 255) / 256), 256, 0, c->stream>>>(u, uf, b.E, K);
    c->prof_end(pk);
  }
  const unsigned nblk = (unsigned)(b.E / NE);
  if (p.system == FR_EULER) {
    pk = c->prof_begin(("hex_div_euler" + sfx).c_str());
    if (wide)
      hex_div_euler_wide<T, DEV, P, NEe, CUR><<<(unsigned)(b.E / NEe), 3 * NEe * N1 * N1, 0, c->stream>>>(
          u, uf, geo, cm, C, r, b.E, b.n, K, (T)p.gamma, p.riemann, R);
    else if constexpr (wide_most < kAnyBlocks)
      hex_div_euler<T, DEV, P, NE, CUR><<<nblk, NT, 0, c->stream>>>(u, uf, geo, cm, C, r, b.E, b.n, K, (T)p.gamma,
                                                                     p.riemann, R);
    c->prof_end(pk);
  } else {
    pk = c->prof_begin(("hex_grad_vf" + sfx).c_str());
    using GC = HexGradCfg<T, P>;
    hex_grad<T, DEV, P, GC::NE, GC::KT, CUR><<<(unsigned)(b.E / GC::NE), GC::NE * N1 * N1 * GC::KT, 0, c->stream>>>(
        u, uf, geo, cm, C, grad, gradf, b.E, K, (T)p.gamma, (T)p.mu, (T)p.prandtl, (T)p.ldg_beta, sm, R);
    c->prof_end(pk);
    T* fc = (T*)b.fc;
    const int64_t face_threads = b.E * 6 * N1 * N1;
    pk = c->prof_begin(("hex_face_vf" + sfx).c_str());
    hex_face_ns<T, DEV, P, CUR><<<(unsigned)((face_threads + 255) / 256), 256, 0, c->stream>>>(
        uf, gradf, geo, cm, C, fc, b.E, b.n, K, (T)p.gamma, (T)p.ldg_beta, (T)p.ldg_tau, p.riemann, sm, R);
    c->prof_end(pk);
    constexpr int NE2 = DivNsCfg<T, P>::NE;
    pk = c->prof_begin(("hex_div_vf" + sfx).c_str());
    // f~_3 of a column in registers except for FP64 at p = 4 (all of f~ in LDS there)
    if constexpr (P <= 3 || sizeof(T) == 4)
      hex_div_ns<T, DEV, P, NE2, CUR><<<(unsigned)(b.E / NE2), NE2 * N1 * N1, 0, c->stream>>>(
          u, grad, fc, geo, cm, r, b.E, b.n, K, (T)p.gamma, R);
    else
      hex_div_ns_lds<T, DEV, P, NE2, CUR><<<(unsigned)(b.E / NE2), NE2 * N1 * N1, 0, c->stream>>>(
          u, grad, fc, geo, cm, r, b.E, b.n, K, (T)p.gamma, R);
    c->prof_end(pk);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(c, FR_ERR_DEVICE, std::string("hex kernel launch: ") + hipGetErrorString(e));
  return FR_OK;
}

// CUR: curved tetrahedra, the metric stored per solution point (b.cmet) in place of the
// per-element terms.
template <typename T, bool DEV, bool CUR>
fr_status tet_rhs(fr_ctx c, DevBlock& b, const T* u, T* r) {
  Conn C{b.nbr_elem, b.nbr_info, c->perm, c->host.perm_stride};
  const fr_params& p = c->prm;
  TetDev<T> O;
  O.src = c->tet_src;
  O.pfp = c->tet_src + 60;
  O.slot = c->tet_src + 60 + 35 * 4;
  O.psrc = (const uint8_t*)(c->tet_src + 60 + 35 * 4 + TET_MP);
  for (int f = 0; f < 4; ++f)
    for (int k = 0; k < 3; ++k) O.nref[f][k] = (T)c->host.tet.nref[f][k];
  const RefState<T> R = ref_of<T>(p);
  const T* geo = (const T*)(CUR ? b.cmet : b.geo_t);
  static const std::string sfx = std::string(CUR ? "_cur" : "") + (sizeof(T) == 8 ? "" : "_f32");
  const int sm = side_mode_of(p.ldg_beta);
  const unsigned div_grid = (unsigned)(b.E / TDIV_NE);   // one 16-element tile per block
  const T* opT = (const T*)c->tet_opT;
  const tet_s4 *opH = (const tet_s4*)c->tet_opH, *opL = opH ? opH + TET_MP * TET_KP16 / 4 : nullptr;
  const tet_s4 *ogH = (const tet_s4*)c->tet_ogH, *ogL = ogH ? ogH + TGR_M * TGR_K / 4 : nullptr;
  // BF16x3 contractions: only in the FP32 form (T = float) when asked for
  constexpr bool can_bf3 = sizeof(T) == 4;
  const bool bf3 = can_bf3 && c->prm.precision == FR_FP32_BF16X3;
  int pk;
  const T zero = T(0);
  if (p.system == FR_EULER) {
    pk = c->prof_begin(("tet_div_euler" + sfx).c_str());
    if (bf3)
      tet_div<T, DEV, false, can_bf3, false, CUR><<<div_grid, tdiv_nt<T>(), 0, c->stream>>>(
          u, nullptr, nullptr, geo, C, O, opT, opH, opL, r, b.E, b.n, (T)p.gamma, zero, zero, zero, zero, p.riemann, 0,
          R);
    else
      tet_div<T, DEV, false, false, false, CUR><<<div_grid, tdiv_nt<T>(), 0, c->stream>>>(
          u, nullptr, nullptr, geo, C, O, opT, opH, opL, r, b.E, b.n, (T)p.gamma, zero, zero, zero, zero, p.riemann, 0,
          R);
    c->prof_end(pk);
  } else {
    // one-sided LDG (beta = +-1/2): the gradient kernel also forms the common fluxes, once
    // per pair, and the divergence reads them (FP64, 24,480 tetrahedra: gradient 86 -> 105 us,
    // divergence 137 -> 76).  Not for FP64 curved elements, whose two sides' stored normals
    // agree to rounding only: one side's unit normal on both moved the low-Mach residual
    // by 1e-9, beyond its rounding floor
    constexpr bool can_fc = tet_can_pair(sizeof(T) == 4, CUR);
    const bool fc = sm != 0 && can_fc;
    T* fcb = (T*)b.fc;
    const T gam = (T)p.gamma, mu = (T)p.mu, pr = (T)p.prandtl, beta = (T)p.ldg_beta, tau = (T)p.ldg_tau;
    const T* ogT = (const T*)c->tet_ogT;
    pk = c->prof_begin(("tet_grad" + sfx).c_str());
#define FR_TET_GRAD(BF, FCX)                                                                                   \
  tet_grad_mma<T, DEV, BF, FCX, CUR><<<div_grid, tgr_nt<T, FCX>(), 0, c->stream>>>(u, geo, C, O, ogT, ogH, ogL, (T*)b.grad, fcb, \
                                                                    b.E, b.n, beta, sm, gam, mu, pr, tau,       \
                                                                    p.riemann, R)
    if (bf3) {
      if (fc) FR_TET_GRAD(can_bf3, can_fc); else FR_TET_GRAD(can_bf3, false);
    } else {
      if (fc) FR_TET_GRAD(false, can_fc); else FR_TET_GRAD(false, false);
    }
#undef FR_TET_GRAD
    c->prof_end(pk);
    pk = c->prof_begin(("tet_div_ns" + sfx).c_str());
#define FR_TET_DIV(BF, FCX)                                                                                     \
  tet_div<T, DEV, true, BF, FCX, CUR><<<div_grid, tdiv_nt<T>(), 0, c->stream>>>(u, (const T*)b.grad, fcb, geo, C, O, opT, opH, \
                                                                     opL, r, b.E, b.n, gam, mu, pr, beta, tau,   \
                                                                     p.riemann, sm, R)
    if (bf3) {
      if (fc) FR_TET_DIV(can_bf3, can_fc); else FR_TET_DIV(can_bf3, false);
    } else {
      if constexpr (sizeof(T) == 8 && !CUR) {
        if (fc)
          tet_div_fv<T><<<div_grid, 256, 0, c->stream>>>(u, (const T*)b.grad, fcb, geo, C, O, opT, r, b.E, b.n, gam, sm,
                                                         R);
        else
          FR_TET_DIV(false, false);
      } else {
        if (fc) FR_TET_DIV(false, can_fc); else FR_TET_DIV(false, false);
      }
    }
#undef FR_TET_DIV
    c->prof_end(pk);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(c, FR_ERR_DEVICE, std::string("tet kernel launch: ") + hipGetErrorString(e));
  return FR_OK;
}

// Pyramids: traces, then (Navier--Stokes) the LDG gradient, then the corrected divergence.
template <typename T, bool DEV>
fr_status pyr_rhs(fr_ctx c, DevBlock& b, const T* u, T* r) {
  Conn C{b.nbr_elem, b.nbr_info, c->perm, c->host.perm_stride};
  const fr_params& p = c->prm;
  const PyrOps& Y = c->host.pyr;
  PyrK<T> K;
  for (int f = 0; f <= 5; ++f) K.face_off[f] = Y.face_off[f];
  for (int f = 0; f < 5; ++f) for (int k = 0; k < 3; ++k) K.nref[f][k] = (T)Y.nref[f][k];
  const T* ops = (const T*)c->pyr_ops;
  PyrOpsDev<T> O{ops, ops + PY_NSP * PY_NFP, ops + PY_NSP * PY_NFP + 3 * PY_NSP * PY_NSP};
  const RefState<T> R = ref_of<T>(p);
  const T* geo = (const T*)b.geo_t;
  T* uf = (T*)b.uf;
  static const std::string sfx = sizeof(T) == 8 ? "" : "_f32";
  if (b.E % 64 != 0) return fail(c, FR_ERR_STATE, "pyramid block not padded to 64 elements");
  const T gam = (T)p.gamma, mu = (T)p.mu, pr = (T)p.prandtl, beta = (T)p.ldg_beta, tau = (T)p.ldg_tau;
  const int sm = side_mode_of(p.ldg_beta);
  // the matrix-core form: Euler, and Navier--Stokes with a one-sided switch (a two-sided
  // common flux needs both sides' gradient traces, which only the general form stores)
  const T* mo = ops + 2 * PY_NSP * PY_NFP + 3 * PY_NSP * PY_NSP;
  const PymOps<T> Q{mo, mo + PYM_KP * PYM_FM, mo + PYM_KP * PYM_FM + 3 * PYM_KP * PYM_M};
  const unsigned nb16 = (unsigned)(b.E / PYM_NE);
  int pk = c->prof_begin(("pyr_trace" + sfx).c_str());
  pyr_trace_mma<T><<<nb16, 64 * PYM_FT, 0, c->stream>>>(u, uf, b.E, Q);
  c->prof_end(pk);
  if (p.system == FR_EULER) {
    pk = c->prof_begin(("pyr_div_euler" + sfx).c_str());
    pyr_div_mma<T, DEV, false><<<nb16, PYM_NT, 0, c->stream>>>(u, uf, nullptr, nullptr, geo, C, Q, K, r, b.E, b.n, gam,
                                                               0, p.riemann, R);
    c->prof_end(pk);
  } else if (sm != 0) {
    T* fv = (T*)b.grad;
    T* fc = (T*)b.fc;
    pk = c->prof_begin(("pyr_grad" + sfx).c_str());
    pyr_grad_mma<T, DEV><<<nb16, PYM_NT, 0, c->stream>>>(u, uf, geo, C, Q, K, fv, fc, b.E, sm, gam, mu, pr, tau,
                                                         p.riemann, R);
    c->prof_end(pk);
    pk = c->prof_begin(("pyr_div_ns" + sfx).c_str());
    pyr_div_mma<T, DEV, true><<<nb16, PYM_NT, 0, c->stream>>>(u, uf, fv, fc, geo, C, Q, K, r, b.E, b.n, gam, sm,
                                                              p.riemann, R);
    c->prof_end(pk);
  } else {
    const unsigned nblk = (unsigned)(b.E / py_ne<T>());
    T* grad = (T*)b.grad;
    T* gradf = (T*)b.gradf;
    pk = c->prof_begin(("pyr_grad" + sfx).c_str());
    pyr_grad<T><<<nblk, PY_NT, 0, c->stream>>>(u, uf, geo, C, O, K, grad, gradf, b.E, beta);
    c->prof_end(pk);
    pk = c->prof_begin(("pyr_div_ns" + sfx).c_str());
    pyr_div<T, DEV><<<nblk, py_nt<T>(), 0, c->stream>>>(u, uf, grad, gradf, geo, C, O, K, r, b.E, gam, mu, pr, beta,
                                                        tau, p.riemann, R);
    c->prof_end(pk);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(c, FR_ERR_DEVICE, std::string("pyramid kernel launch: ") + hipGetErrorString(e));
  return FR_OK;
}

template <typename T, bool DEV>
fr_status rhs_t(fr_ctx c, const T* u, void* const* r) {
  for (size_t bi = 0; bi < c->blocks.size(); ++bi) {
    DevBlock& b = c->blocks[bi];
    const T* ub = u + b.native_off;
    T* rb = (T*)r[bi];
    fr_status s = FR_OK;
    if (b.etype == FR_HEX) {
      switch (c->prm.order) {
        case 1: s = b.cmet ? hex_rhs_p<T, DEV, 1, true>(c, b, ub, rb) : hex_rhs_p<T, DEV, 1, false>(c, b, ub, rb); break;
        case 2: s = b.cmet ? hex_rhs_p<T, DEV, 2, true>(c, b, ub, rb) : hex_rhs_p<T, DEV, 2, false>(c, b, ub, rb); break;
        case 3: s = b.cmet ? hex_rhs_p<T, DEV, 3, true>(c, b, ub, rb) : hex_rhs_p<T, DEV, 3, false>(c, b, ub, rb); break;
        case 4: s = b.cmet ? hex_rhs_p<T, DEV, 4, true>(c, b, ub, rb) : hex_rhs_p<T, DEV, 4, false>(c, b, ub, rb); break;
        default: s = fail(c, FR_ERR_UNSUPPORTED, "order");
      }
    } else if (b.etype == FR_PYR) {
      s = pyr_rhs<T, DEV>(c, b, ub, rb);
    } else {
      s = b.cmet ? tet_rhs<T, DEV, true>(c, b, ub, rb) : tet_rhs<T, DEV, false>(c, b, ub, rb);
    }
    if (s != FR_OK) return s;
  }
  return FR_OK;
}

constexpr size_t kMaxBlocks = 2;

// RHS of the context's precision on its native state, block i of it into r[i].
fr_status rhs_blocks(fr_ctx c, const void* u, void* const* r) {
  if (c->prm.precision != FR_FP64) return rhs_t<float, true>(c, (const float*)u, r);
  return rhs_t<double, false>(c, (const double*)u, r);
}

size_t native_size(fr_ctx c) { return c->prm.precision != FR_FP64 ? sizeof(float) : sizeof(double); }

// The same into one native array.
fr_status rhs_native(fr_ctx c, const void* u, void* r) {
  void* rb[kMaxBlocks] = {};
  for (size_t i = 0; i < c->blocks.size(); ++i) rb[i] = (char*)r + c->blocks[i].native_off * native_size(c);
  return rhs_blocks(c, u, rb);
}

RefVec refvec(const fr_params& p) {
  RefVec r;
  for (int i = 0; i < 5; ++i) r.v[i] = p.u_ref[i];
  return r;
}


// ------------------------------------------------------------ entropy filter
FiltK filtk_of(const HexOps& H) {
  FiltK k;
  std::memset(&k, 0, sizeof(k));
  for (int a = 0; a < 5; ++a) {
    k.lm[a] = H.lm[a];
    k.lp[a] = H.lp[a];
    for (int m = 0; m < 5; ++m) { k.Vm[a][m] = H.Vm[a][m]; k.Vmi[a][m] = H.Vmi[a][m]; }
  }
  for (int m = 0; m < H.n1; ++m) {
    const double nm = std::sqrt((2.0 * m + 1.0) / 2.0);
    k.Pe[0][m] = nm * ((m % 2) ? -1.0 : 1.0);
    k.Pe[1][m] = nm;
  }
  return k;
}

FiltPrm filtprm_of(const fr_params& p, int order) {
  FiltPrm f;
  f.gamma = p.gamma;
  f.eps_rho = p.filt_eps_rho;
  f.eps_p = p.filt_eps_p;
  f.eps_s = p.filt_eps_s;
  f.zeta_max = p.filt_zeta_max_coef * order * order;
  f.n_bits = p.filt_bits;
  return f;
}

fr_status filter_alloc(fr_ctx c) {
  for (auto& b : c->blocks)
    if (b.etype == FR_PYR)
      return fail(c, FR_ERR_UNSUPPORTED, "the entropy filter and its learned warm start have no pyramid form");
  if (c->f_k) return FR_OK;
  bool has_tet = false;
  for (auto& b : c->blocks) has_tet = has_tet || b.etype == FR_TET;
  if (has_tet && !c->tet_ftab) {
    // V^T, V^{-1} transposed, normalised weights, check-point multiplicities
    const TetOps& T = c->host.tet;
    std::vector<double> tab(TF_LEN);
    double wsum = 0;
    for (int z = 0; z < TF_NSP; ++z) wsum += T.weights[z];
    for (int m = 0; m < TF_NSP; ++m) {
      if (T.deg[m] != tet_mode_deg(m)) return fail(c, FR_ERR_STATE, "tetrahedral modes not graded by degree");
      for (int z = 0; z < TF_NSP; ++z) {
        tab[TF_VT + m * TF_NSP + z] = T.V[z][m];
        tab[TF_VIT + z * TF_NSP + m] = T.Vinv[m][z];
      }
    }
    for (int z = 0; z < TF_NSP; ++z) {
      tab[TF_W + z] = T.weights[z] / wsum;
      tab[TF_MULT + z] = 1.0;
    }
    for (int f = 0; f < TetOps::nfp; ++f) tab[TF_MULT + T.fp_src[f]] += 1.0;
    if (dalloc(c, &c->tet_ftab, TF_LEN)) return FR_ERR_ALLOC;
    HIP_TRY(c, hipMemcpy(c->tet_ftab, tab.data(), TF_LEN * sizeof(double), hipMemcpyHostToDevice));
  }
  const int64_t n = c->n_elem_total;
  for (auto& b : c->blocks)
    if (dalloc(c, &b.sown, b.E) || dalloc(c, &b.smin, b.E) || dalloc(c, &b.f_det, b.n) ||
        dalloc(c, &b.f_list, b.n) || dalloc(c, &b.f_cnt, FILT_SLOTS))
      return FR_ERR_ALLOC;
  if (dalloc(c, &c->f_k, n) || dalloc(c, &c->f_evals, n) || dalloc(c, &c->f_flag, n) ||
      dalloc(c, &c->f_feat, n * 16) || dalloc(c, &c->f_khat, n))
    return FR_ERR_ALLOC;
  return FR_OK;
}

// An RK4 stage update fused into the filter's detection pass (see RkStageSrc): the
// pass forms the stage state (or the new state) while checking it.
struct StageFuse {
  int stage = 0;                // 0..3; the last one updates u in place
  double b = 0, c = 0;          // accumulator and stage coefficients (times dt)
  bool k32 = false;             // increments (and s32) FP32: the FP32 form
  double* u = nullptr;          // u_n, or the state updated in place (last stage)
  double* s64 = nullptr;        // FP64 stage state written in full (FP64 form) or null
  float* s32 = nullptr;         // FP32 deviation of the stage state (FP32 form) or null
  double* cand64 = nullptr;     // FP64 stage state of the candidates only (FP32 form) or null
  double b1 = 0, b2 = 0;        // FP32 form: the coefficients of the kept increments (times dt)
};

// Increment of RK stage s (0..3) of a block.  FP64: 0 shares RK4's accumulator, which RK4 writes
// before it reads it (the embedded pair keeps all of them, RK4 uses 3 alone).
char* rk_inc(fr_ctx c, const DevBlock& b, int s) {
  const int64_t o = b.native_off, len = (int64_t)b.nsp * 5 * b.E;
  if (s == 3) return (char*)c->rk_k + o * native_size(c);
  if (c->prm.precision != FR_FP64) return (char*)((float*)c->rk_kk + 3 * o + s * len);
  return (char*)(s == 0 ? c->rk_acc + o : (double*)c->rk_kk + (s - 1) * c->native_len + o);
}

// FP64 accumulator of a block.  In the FP32 form only filtered hexahedra keep one, over the
// increments that they do not keep (two FP32 arrays).
double* rk_accum(fr_ctx c, const DevBlock& b) {
  return c->prm.precision != FR_FP64 ? (double*)((float*)c->rk_kk + 3 * b.native_off) : c->rk_acc + b.native_off;
}

template <typename KT>
RkStageSrc<KT> stage_src(fr_ctx c, const StageFuse& z, const DevBlock& b) {
  const int64_t o = b.native_off;
  RkStageSrc<KT> s{z.u + o, (const KT*)rk_inc(c, b, 3), rk_accum(c, b), z.s64 ? z.s64 + o : nullptr,
                   z.s32 ? z.s32 + o : nullptr, z.b, z.c, z.stage == 0 ? 0 : (z.stage < 3 ? 1 : 2), {0, 0, 0, 0, 0}};
  for (int v = 0; v < 5; ++v) s.ref[v] = c->prm.u_ref[v];
  return s;
}

template <int P>
void hex_smin_p(fr_ctx c, DevBlock& b, const double* uprev) {
  const FiltK K = filtk_of(c->host.hex);
  const int g = (int)((b.n + 255) / 256);
  unsigned long long* sown = (unsigned long long*)b.sown;
  int pk = c->prof_begin("filter_smin");
  hex_sown<P><<<(unsigned)(b.E / HexTileCfg<P>::NE), HexTileCfg<P>::NT, 0, c->stream>>>(
      uprev + b.native_off, sown, b.E, b.n, K, c->prm.gamma);
  elem_smin<<<g, 256, 0, c->stream>>>(sown, b.nbr_elem, b.nfaces, b.smin, b.E, b.n, b.f_det, b.f_cnt);
  c->prof_end(pk);
}

// The candidate list of the current filter call on block b.
CandList cand_list(fr_ctx c, const DevBlock& b) {
  return CandList{b.f_list, b.f_cnt + c->f_slot, b.f_det, c->f_k + b.elem_off, c->f_evals + b.elem_off,
                  c->f_slot + 1, b.n};
}

// Candidates of the search: detection at zeta = 0 into b.f_list / count b.f_cnt[slot];
// untouched elements get k = 0 and one evaluation.
template <int P>
void hex_candidates_p(fr_ctx c, DevBlock& b, const double* u, const StageFuse* fz = nullptr) {
  const FiltK K = filtk_of(c->host.hex);
  const FiltPrm F = filtprm_of(c->prm, P);
  const CandList L = cand_list(c, b);
  int pk = c->prof_begin(fz ? "rk4_stage_filter_detect_hex" : "filter_detect");
  if constexpr (P == 4) {
    // p = 4: a tile holds only 8 elements, so the tiled pass would move its rows in
    // 64-byte segments; one wave per (64-element tile, column) reads whole 512-byte rows
    // and the line ends through L2 (0.78 -> 0.72 ms per stage on the mixed workload).
    // At p <= 3 (16-64 elements a tile) the tiled pass is faster (1.43 against 1.63 ms
    // per step on the 48^3 p = 3 shock).
    const unsigned g = (unsigned)((b.E / 64 * (P + 1) * (P + 1) + 3) / 4);
    if (!fz)
      hex_filter_detect_lines<P, PlainSrc><<<g, 256, 0, c->stream>>>(PlainSrc{u + b.native_off}, b.smin, b.E,
                                                                     b.n, K, F, L);
    else if (fz->k32)
      hex_filter_detect_lines<P, RkStageSrc<float>><<<g, 256, 0, c->stream>>>(stage_src<float>(c, *fz, b),
                                                                              b.smin, b.E, b.n, K, F, L);
    else
      hex_filter_detect_lines<P, RkStageSrc<double>><<<g, 256, 0, c->stream>>>(stage_src<double>(c, *fz, b),
                                                                               b.smin, b.E, b.n, K, F, L);
  } else {
    const unsigned g = (unsigned)(b.E / HexTileCfg<P>::NE);
    if (!fz)
      hex_filter_detect<P, PlainSrc><<<g, HexTileCfg<P>::NT, 0, c->stream>>>(PlainSrc{u + b.native_off}, b.smin,
                                                                             b.E, b.n, K, F, L, nullptr);
    else if (fz->k32)
      hex_filter_detect<P, RkStageSrc<float>><<<g, HexTileCfg<P>::NT, 0, c->stream>>>(
          stage_src<float>(c, *fz, b), b.smin, b.E, b.n, K, F, L,
          fz->cand64 ? fz->cand64 + b.native_off : nullptr);
    else
      hex_filter_detect<P, RkStageSrc<double>><<<g, HexTileCfg<P>::NT, 0, c->stream>>>(
          stage_src<double>(c, *fz, b), b.smin, b.E, b.n, K, F, L,
          fz->cand64 ? fz->cand64 + b.native_off : nullptr);
  }
  if (P == 4 && fz && fz->cand64 && fz->k32)
    k_cand_stage<float><<<(unsigned)std::max<int64_t>(1, std::min<int64_t>(b.n, 4096)), 256, 0, c->stream>>>(
        stage_src<float>(c, *fz, b), b.f_list, b.f_cnt + c->f_slot, b.nsp * 5, b.E, fz->cand64 + b.native_off);
  c->prof_end(pk);
}

// Grid of the per-candidate filter kernels: FW candidates (waves) per block.
inline unsigned list_grid(const DevBlock& b, int fw) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((b.n + fw - 1) / fw, 2048));
}

// Features (and the exact troubled flag) of the candidates of b.
template <int P>
void hex_features_p(fr_ctx c, DevBlock& b, const double* u) {
  const FiltK K = filtk_of(c->host.hex);
  const FiltPrm F = filtprm_of(c->prm, P);
  const int64_t o = b.elem_off;
  k_fill_i32<<<grid_for(b.n, 256), 256, 0, c->stream>>>(c->f_flag + o, b.n, 0);
  constexpr int FW = HexFW<P>::value;
  hex_features<P><<<list_grid(b, FW), 64 * FW, 0, c->stream>>>(u + b.native_off, b.smin, b.E, b.f_list, b.f_cnt + c->f_slot, K, F,
                                                       c->f_flag + o, c->f_feat + o * 16);
}

template <int P>
void hex_filter_p(fr_ctx c, DevBlock& b, double* u, int mode, float* u32, const StageFuse* fz) {
  constexpr int FW = HexFW<P>::value;
  const FiltK K = filtk_of(c->host.hex);
  const FiltPrm F = filtprm_of(c->prm, P);
  const int64_t o = b.elem_off;
  Dev32 s32{u32 ? u32 + b.native_off : nullptr, {0, 0, 0, 0, 0}};
  for (int v = 0; v < 5; ++v) s32.ref[v] = c->prm.u_ref[v];
  hex_candidates_p<P>(c, b, u, fz);
  int pk;
  if (mode == 1) {
    pk = c->prof_begin("filter_search_learned");
    hex_filter_learned<P><<<list_grid(b, FW), 64 * FW, 0, c->stream>>>(
        u + b.native_off, b.smin, b.E, b.f_list, b.f_cnt + c->f_slot, K, F, c->m_w, c->m_scale, c->f_k + o,
        c->f_evals + o, s32);
  } else {
    pk = c->prof_begin("filter_search_plain");
    hex_filter<P><<<list_grid(b, FW), 64 * FW, 0, c->stream>>>(u + b.native_off, b.smin, b.E, b.f_list,
                                                               b.f_cnt + c->f_slot, K, F, c->f_k + o, c->f_evals + o, s32);
  }
  c->prof_end(pk);
}


void tet_smin(fr_ctx c, DevBlock& b, const double* uprev) {
  const int g = (int)((b.n + 255) / 256);
  unsigned long long* sown = (unsigned long long*)b.sown;
  int pk = c->prof_begin("filter_smin");
  tet_sown<<<(unsigned)(b.E / 64), TF_NT, 0, c->stream>>>(uprev + b.native_off, sown, b.E, b.n, c->prm.gamma);
  elem_smin<<<g, 256, 0, c->stream>>>(sown, b.nbr_elem, b.nfaces, b.smin, b.E, b.n, b.f_det, b.f_cnt);
  c->prof_end(pk);
}

void tet_candidates(fr_ctx c, DevBlock& b, const double* u, const StageFuse* fz = nullptr) {
  const FiltPrm F = filtprm_of(c->prm, c->prm.order);
  const CandList L = cand_list(c, b);
  int pk = c->prof_begin(fz ? "rk4_stage_filter_detect_tet" : "filter_detect");
  const unsigned gE = (unsigned)(b.E / 64);
  if (!fz)
    tet_filter_detect<PlainSrc><<<gE, TF_NT, 0, c->stream>>>(PlainSrc{u + b.native_off}, b.smin, b.E, b.n, F, L,
                                                           nullptr);
  else if (fz->k32) {
    const int64_t o = b.native_off;
    auto inc = [&](int s) { return (const float*)rk_inc(c, b, s); };
    RkKeepSrc src{fz->u + o, inc(fz->stage), inc(0), inc(1), inc(2),
                  fz->s32 + o, fz->b1, fz->b2, fz->c, fz->stage == 3, {0, 0, 0, 0, 0}};
    for (int v = 0; v < 5; ++v) src.ref[v] = c->prm.u_ref[v];
    tet_filter_detect<RkKeepSrc><<<gE, TF_NT, 0, c->stream>>>(src, b.smin, b.E, b.n, F, L,
                                                              fz->cand64 ? fz->cand64 + o : nullptr);
  }
  else
    tet_filter_detect<RkStageSrc<double>><<<gE, TF_NT, 0, c->stream>>>(
        stage_src<double>(c, *fz, b), b.smin, b.E, b.n, F, L,
        fz->cand64 ? fz->cand64 + b.native_off : nullptr);
  c->prof_end(pk);
}

void tet_features_b(fr_ctx c, DevBlock& b, const double* u) {
  const FiltPrm F = filtprm_of(c->prm, c->prm.order);
  const int64_t o = b.elem_off;
  k_fill_i32<<<grid_for(b.n, 256), 256, 0, c->stream>>>(c->f_flag + o, b.n, 0);
  tet_features<<<list_grid(b, 4), 256, 0, c->stream>>>(u + b.native_off, b.smin, b.E, b.f_list, b.f_cnt + c->f_slot,
                                                         c->tet_ftab, F, c->f_flag + o, c->f_feat + o * 16);
}

void tet_filter_b(fr_ctx c, DevBlock& b, double* u, int mode, float* u32, const StageFuse* fz) {
  const FiltPrm F = filtprm_of(c->prm, c->prm.order);
  const int64_t o = b.elem_off;
  Dev32 s32{u32 ? u32 + b.native_off : nullptr, {0, 0, 0, 0, 0}};
  for (int v = 0; v < 5; ++v) s32.ref[v] = c->prm.u_ref[v];
  tet_candidates(c, b, u, fz);
  int pk;
  if (mode == 1) {
    pk = c->prof_begin("filter_search_learned");
    tet_filter_learned<<<list_grid(b, 4), 256, 0, c->stream>>>(u + b.native_off, b.smin, b.E, b.f_list,
                                                                 b.f_cnt + c->f_slot, c->tet_ftab, F, c->m_w, c->m_scale,
                                                                 c->f_k + o, c->f_evals + o, s32);
  } else {
    pk = c->prof_begin("filter_search_plain");
    tet_filter<<<list_grid(b, 4), 256, 0, c->stream>>>(u + b.native_off, b.smin, b.E, b.f_list, b.f_cnt + c->f_slot,
                                                         c->tet_ftab, F, c->f_k + o, c->f_evals + o, s32);
  }
  c->prof_end(pk);
}

fr_status compute_smin(fr_ctx c, const double* uprev) {
  c->f_slot = -1;
  for (auto& b : c->blocks) {
    if (b.etype == FR_TET) {
      tet_smin(c, b, uprev);
      continue;
    }
    switch (c->prm.order) {
      case 1: hex_smin_p<1>(c, b, uprev); break;
      case 2: hex_smin_p<2>(c, b, uprev); break;
      case 3: hex_smin_p<3>(c, b, uprev); break;
      case 4: hex_smin_p<4>(c, b, uprev); break;
    }
  }
  HIP_TRY(c, hipGetLastError());
  return FR_OK;
}

fr_status collect_rows(fr_ctx c, const double* u);
fr_status apply_filter(fr_ctx c, double* u, int mode, float* u32 = nullptr, const StageFuse* fz = nullptr);

// Filter the FP64 native state u in place; with u32 (the FP32 form's stage buffer) the
// filtered elements' FP32 deviations are rewritten there as well.  With fz the
// detection pass first performs that RK stage update (u is then the buffer the search
// works on: the full FP64 stage state, the candidates' copy, or the new state).
fr_status apply_filter(fr_ctx c, double* u, int mode, float* u32, const StageFuse* fz) {
  if (c->collecting) {
    if (fz) return fail(c, FR_ERR_STATE, "training-data collection needs the stage state before the filter");
    fr_status st = collect_rows(c, u);
    if (st) return st;
  }
  if ((++c->f_slot) >= FILT_SLOTS) return fail(c, FR_ERR_STATE, "more filter calls per s_min pass than counters");
  for (auto& b : c->blocks) {
    if (b.etype == FR_TET) {
      tet_filter_b(c, b, u, mode, u32, fz);
      continue;
    }
    switch (c->prm.order) {
      case 1: hex_filter_p<1>(c, b, u, mode, u32, fz); break;
      case 2: hex_filter_p<2>(c, b, u, mode, u32, fz); break;
      case 3: hex_filter_p<3>(c, b, u, mode, u32, fz); break;
      case 4: hex_filter_p<4>(c, b, u, mode, u32, fz); break;
    }
  }
  HIP_TRY(c, hipGetLastError());
  return FR_OK;
}

__global__ void k_gather_features(const float* __restrict__ feat, const int32_t* __restrict__ kk,
                                  const int32_t* __restrict__ idx, int64_t n, float* __restrict__ x,
                                  int32_t* __restrict__ elem, int32_t* __restrict__ kout) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t e = idx[i];
  for (int f = 0; f < 16; ++f) x[i * 16 + f] = feat[(int64_t)e * 16 + f];
  if (elem) elem[i] = e;
  if (kout) kout[i] = kk[e];
}

// Features and plain-search targets of the troubled elements of u (entropy bound
// from the current s_min), appended to the collection buffers.
template <int P>
void hex_candidate_features_p(fr_ctx c, DevBlock& b, const double* u) {
  hex_candidates_p<P>(c, b, u);
  hex_features_p<P>(c, b, u);
}

fr_status candidate_features(fr_ctx c, const double* u) {
  if ((++c->f_slot) >= FILT_SLOTS) return fail(c, FR_ERR_STATE, "more filter calls per s_min pass than counters");
  for (auto& b : c->blocks) {
    if (b.etype == FR_TET) {
      tet_candidates(c, b, u);
      tet_features_b(c, b, u);
      continue;
    }
    switch (c->prm.order) {
      case 1: hex_candidate_features_p<1>(c, b, u); break;
      case 2: hex_candidate_features_p<2>(c, b, u); break;
      case 3: hex_candidate_features_p<3>(c, b, u); break;
      case 4: hex_candidate_features_p<4>(c, b, u); break;
    }
  }
  HIP_TRY(c, hipGetLastError());
  return FR_OK;
}

fr_status collect_rows(fr_ctx c, const double* u) {
  fr_status cs = candidate_features(c, u);
  if (cs) return cs;
  HIP_TRY(c, hipMemcpyAsync(c->f_copy, u, c->native_len * sizeof(double), hipMemcpyDeviceToDevice, c->stream));
  c->collecting = false;
  fr_status st = apply_filter(c, c->f_copy, 0);
  c->collecting = true;
  if (st) return st;
  std::vector<int32_t> flag(c->n_elem_total);
  HIP_TRY(c, hipMemcpyAsync(flag.data(), c->f_flag, flag.size() * 4, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  std::vector<int32_t> idx;
  for (size_t i = 0; i < flag.size(); ++i) if (flag[i]) idx.push_back((int32_t)i);
  c->col_seen += (int64_t)idx.size();
  const int64_t m = std::min<int64_t>((int64_t)idx.size(), c->col_cap - c->col_n);
  if (m > 0) {
    int32_t* didx = nullptr;
    if (dalloc(c, &didx, m)) return FR_ERR_ALLOC;
    HIP_TRY(c, hipMemcpyAsync(didx, idx.data(), m * 4, hipMemcpyHostToDevice, c->stream));
    k_gather_features<<<(unsigned)((m + 255) / 256), 256, 0, c->stream>>>(c->f_feat, c->f_k, didx, m,
                                                                          c->col_x + c->col_n * 16, nullptr,
                                                                          c->col_k + c->col_n);
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    (void)hipFree(didx);
    c->col_n += m;
  }
  return FR_OK;
}

fr_status mlp_alloc(fr_ctx c, int batch) {
  if (!c->m_w) {
    if (dalloc(c, &c->m_w, MLP_NP) || dalloc(c, &c->m_m, MLP_NP) || dalloc(c, &c->m_v, MLP_NP) ||
        dalloc(c, &c->m_scale, 2 * MLP_IN) || dalloc(c, &c->m_loss, 1))
      return FR_ERR_ALLOC;
  }
  if (batch > c->m_batch_cap) {
    (void)hipFree(c->m_scratch);
    (void)hipFree(c->m_sqerr);
    if (dalloc(c, &c->m_scratch, (size_t)batch * MLP_SS) || dalloc(c, &c->m_sqerr, batch)) return FR_ERR_ALLOC;
    c->m_batch_cap = batch;
  }
  return FR_OK;
}

}  // namespace

// =============================================================================
extern "C" {

void fr_default_params(fr_params* p) {
  if (!p) return;
  std::memset(p, 0, sizeof(*p));
  p->struct_size = sizeof(fr_params);
  p->system = FR_EULER;
  p->order = 3;
  p->riemann = FR_RUSANOV;
  p->precision = FR_FP64;
  p->gamma = 1.4;
  p->mu = 1.0 / 1600.0;
  p->prandtl = 0.71;
  p->ldg_beta = 0.5;
  p->ldg_tau = 0.1;
  p->u_ref[0] = 1.0;
  p->u_ref[4] = 1.0 / (0.4 * 1.4 * 0.01);
  p->filt_eps_rho = 1e-8;
  p->filt_eps_p = 1e-8;
  p->filt_eps_s = 1e-4;
  p->filt_zeta_max_coef = 40.0;
  p->filt_bits = 20;
}

const char* fr_last_error(fr_ctx ctx) { return ctx ? ctx->err.c_str() : g_thread_err.c_str(); }

void fr_destroy(fr_ctx c) {
  if (!c) return;
  if (c->stream) (void)hipStreamSynchronize(c->stream);
  for (auto& b : c->blocks) {
    if (b.geo_t && b.geo_t != b.geo) (void)hipFree(b.geo_t);
    (void)hipFree(b.geo); (void)hipFree(b.nbr_elem); (void)hipFree(b.nbr_info);
    (void)hipFree(b.uf); (void)hipFree(b.grad); (void)hipFree(b.gradf); (void)hipFree(b.fc);
    (void)hipFree(b.cmet);
    (void)hipFree(b.cpos);
  }
  (void)hipFree(c->perm);
  (void)hipFree(c->g_npos);
  (void)hipFree(c->rk_stage); (void)hipFree(c->rk_acc); (void)hipFree(c->rk_k); (void)hipFree(c->rk_s64);
  (void)hipFree(c->rk_kk);
  (void)hipFree(c->rk_x0); (void)hipFree(c->rk_part);
  (void)hipFree(c->flag);
  (void)hipFree(c->tet_src); (void)hipFree(c->tet_opT); (void)hipFree(c->tet_ogT); (void)hipFree(c->pyr_ops);
  (void)hipFree(c->tet_opH); (void)hipFree(c->tet_ogH); (void)hipFree(c->tet_ftab);
  for (auto& b : c->blocks) {
    (void)hipFree(b.sown); (void)hipFree(b.smin);
    (void)hipFree(b.f_det); (void)hipFree(b.f_list); (void)hipFree(b.f_cnt);
  }
  for (void* q : {(void*)c->f_k, (void*)c->f_evals, (void*)c->f_flag, (void*)c->f_feat, (void*)c->f_khat,
                  (void*)c->f_copy, (void*)c->m_w, (void*)c->m_m, (void*)c->m_v, (void*)c->m_scale,
                  (void*)c->m_loss, (void*)c->m_scratch, (void*)c->m_sqerr, (void*)c->m_idx})
    (void)hipFree(q);
  c->prof_clear();
  delete c;
}

namespace {
fr_status setup_impl(const fr_params* p, int64_t n_vert, const double* xyz, const double* period,
                     int64_t n_elem, const int32_t* etype, const int64_t* enodes, int geo_order,
                     const int64_t* ho_nodes, void* stream, fr_ctx* out) {
  if (!out) return fail(nullptr, FR_ERR_ARG, "out is NULL");
  *out = nullptr;
  if (!p || p->struct_size != sizeof(fr_params)) return fail(nullptr, FR_ERR_ARG, "fr_params missing or struct_size mismatch");
  if (!xyz || !period || !etype || !enodes || n_vert <= 0 || n_elem <= 0) return fail(nullptr, FR_ERR_ARG, "empty mesh or NULL array");
  if (p->system != FR_EULER && p->system != FR_NAVIER_STOKES) return fail(nullptr, FR_ERR_ARG, "system");
  if (p->riemann != FR_RUSANOV && p->riemann != FR_HLLC) return fail(nullptr, FR_ERR_ARG, "riemann");
  if (p->precision != FR_FP64 && p->precision != FR_FP32 && p->precision != FR_FP32_BF16X3)
    return fail(nullptr, FR_ERR_ARG, "precision");
  if (p->precision == FR_FP32_BF16X3 && std::none_of(etype, etype + n_elem, [](int32_t t) { return t == FR_TET; }))
    return fail(nullptr, FR_ERR_UNSUPPORTED,
                "FR_FP32_BF16X3 splits the dense tetrahedral operator products; a mesh without tetrahedra has "
                "none (hexahedra contract 1-D lines on the vector units): use FR_FP32");
  if (p->precision != FR_FP64 && (p->u_ref[1] != 0 || p->u_ref[2] != 0 || p->u_ref[3] != 0 ||
                                  !(p->u_ref[0] > 0) || !(p->u_ref[4] > 0)))
    return fail(nullptr, FR_ERR_ARG, "the FP32 form needs a reference state at rest with rho > 0, E > 0");
  if (!(p->gamma > 1.0)) return fail(nullptr, FR_ERR_ARG, "gamma must exceed 1");
  if (p->filt_bits < 1 || p->filt_bits > 30) return fail(nullptr, FR_ERR_ARG, "filt_bits must be in 1..30");
  if (!(p->filt_zeta_max_coef > 0) || !std::isfinite(p->filt_zeta_max_coef))
    return fail(nullptr, FR_ERR_ARG, "filt_zeta_max_coef must be positive and finite");
  if (!(p->filt_eps_rho >= 0) || !(p->filt_eps_p >= 0) || !(p->filt_eps_s >= 0))
    return fail(nullptr, FR_ERR_ARG, "filter floors and entropy tolerance must be >= 0");
  if (p->elem_order < 0 || p->elem_order > 2) return fail(nullptr, FR_ERR_ARG, "elem_order must be 0, 1 or 2");
  if (p->hex_metric != FR_METRIC_CONSERVATIVE && p->hex_metric != FR_METRIC_CROSS)
    return fail(nullptr, FR_ERR_ARG, "hex_metric must be FR_METRIC_CONSERVATIVE or FR_METRIC_CROSS");
  fr_ctx c = new (std::nothrow) fr_ctx_s();
  if (!c) return fail(nullptr, FR_ERR_ALLOC, "context allocation");
  c->prm = *p;
  c->stream = (hipStream_t)stream;
  c->static_scratch = static_scratch_address();
  int code = 0;
  std::string msg;
  try {
    msg = build_setup(p->order, n_vert, xyz, period, n_elem, etype, enodes, 64, p->elem_order, c->host, code);
    if (msg.empty() && ho_nodes) {
      const bool tets = !c->host.blocks.empty() && c->host.blocks[0].etype == kTet;
      msg = tets ? build_curved_tet(geo_order, p->hex_metric, xyz, ho_nodes, c->host, code)
                 : build_curved_hex(geo_order, p->hex_metric, xyz, ho_nodes, c->host, code);
    }
  } catch (const std::exception& ex) {
    msg = ex.what();
    code = 3;
  }
  if (!msg.empty()) {
    fr_status s = code == 2 ? FR_ERR_MESH : (code == 3 ? FR_ERR_UNSUPPORTED : FR_ERR_ARG);
    delete c;
    return fail(nullptr, s, msg);
  }
  const size_t tsz = p->precision != FR_FP64 ? sizeof(float) : sizeof(double);
  int64_t canon = 0, native = 0;
  auto bail = [&](fr_status s) { std::string m = c->err; fr_destroy(c); return fail(nullptr, s, m); };
  for (auto& hb : c->host.blocks) {
    DevBlock b;
    b.etype = hb.etype; b.n = hb.n; b.E = hb.e_pad; b.nsp = hb.nsp; b.nfp = hb.nfp; b.nfaces = hb.nfaces;
    b.canon_off = canon; b.native_off = native;
    b.elem_off = c->n_elem_total;
    c->n_elem_total += b.n;
    canon += b.n * 5 * b.nsp;
    native += b.E * 5 * b.nsp;
    c->blocks.push_back(b);
    DevBlock& d = c->blocks.back();
    {
      std::vector<int32_t> cp((size_t)d.E, -1);
      for (int64_t i = 0; i < d.n; ++i) cp[i] = hb.canon_pos[i];
      if (dalloc(c, &d.cpos, cp.size())) return bail(FR_ERR_ALLOC);
      if (hipMemcpy(d.cpos, cp.data(), cp.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
        c->err = "upload failed";
        return bail(FR_ERR_DEVICE);
      }
    }
    if (dalloc(c, &d.geo, hb.geo.size()) || dalloc(c, &d.nbr_elem, hb.nbr_elem.size()) ||
        dalloc(c, &d.nbr_info, hb.nbr_info.size()))
      return bail(FR_ERR_ALLOC);
    // what the kernels of this context's form read: traces of u except on tetrahedra (their flux
    // points are solution points); Navier--Stokes: the points' viscous flux (hexahedra 9 values, with
    // once-per-pair common fluxes 12) or gradient (15), the gradient's traces (hexahedra f_v.n, pyramids
    // with a two-sided switch), the common fluxes where they are stored
    const bool is_tet = d.etype == FR_TET, is_hex = d.etype == FR_HEX, ns = p->system == FR_NAVIER_STOKES;
    const bool pair = side_mode_of(p->ldg_beta) != 0 &&
                      (!is_tet || tet_can_pair(tsz == sizeof(float), !hb.cmet.empty()));
    const int64_t rows[4] = {is_tet ? 0 : 5 * d.nfp, !ns ? 0 : d.nsp * (is_hex ? 9 : (pair ? 12 : 15)),
                             !ns || is_tet ? 0 : d.nfp * (is_hex ? 4 : (pair ? 0 : 15)),
                             ns && (is_hex || pair) ? 5 * d.nfp : 0};
    void** const at[4] = {&d.uf, &d.grad, &d.gradf, &d.fc};
    for (int k = 0; k < 4; ++k)
      if (rows[k] && dalloc(c, (char**)at[k], (size_t)(rows[k] * d.E) * tsz)) return bail(FR_ERR_ALLOC);
    d.geo_t = d.geo;
    if (tsz == sizeof(float)) {
      std::vector<float> g32(hb.geo.begin(), hb.geo.end());
      if (dalloc(c, (float**)&d.geo_t, g32.size())) return bail(FR_ERR_ALLOC);
      if (hipMemcpy(d.geo_t, g32.data(), g32.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess) {
        c->err = "upload failed";
        return bail(FR_ERR_DEVICE);
      }
    }
    if (!hb.cmet.empty()) {
      if (tsz == sizeof(float)) {
        std::vector<float> m32(hb.cmet.begin(), hb.cmet.end());
        if (dalloc(c, (float**)&d.cmet, m32.size())) return bail(FR_ERR_ALLOC);
        if (hipMemcpy(d.cmet, m32.data(), m32.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess) {
          c->err = "upload failed";
          return bail(FR_ERR_DEVICE);
        }
      } else {
        if (dalloc(c, (double**)&d.cmet, hb.cmet.size())) return bail(FR_ERR_ALLOC);
        if (hipMemcpy(d.cmet, hb.cmet.data(), hb.cmet.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) {
          c->err = "upload failed";
          return bail(FR_ERR_DEVICE);
        }
      }
    }
    if (hipMemcpy(d.geo, hb.geo.data(), hb.geo.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(d.nbr_elem, hb.nbr_elem.data(), hb.nbr_elem.size() * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(d.nbr_info, hb.nbr_info.data(), hb.nbr_info.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
      c->err = "upload failed";
      return bail(FR_ERR_DEVICE);
    }
  }
  c->canon_len = canon;
  c->native_len = native;
  {
    std::vector<int32_t> gn((size_t)c->n_elem_total);
    c->h_cpos.assign((size_t)c->n_elem_total, 0);
    for (size_t bi = 0; bi < c->blocks.size(); ++bi) {
      const Block& hb = c->host.blocks[bi];
      const int64_t o = c->blocks[bi].elem_off;
      for (int64_t i = 0; i < hb.n; ++i) {
        c->h_cpos[o + i] = (int32_t)(o + hb.canon_pos[i]);
        gn[o + hb.canon_pos[i]] = (int32_t)(o + i);
      }
    }
    if (dalloc(c, &c->g_npos, gn.size())) return bail(FR_ERR_ALLOC);
    if (hipMemcpy(c->g_npos, gn.data(), gn.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
      c->err = "upload failed";
      return bail(FR_ERR_DEVICE);
    }
  }
  if (dalloc(c, &c->perm, c->host.orient_perm.size()) || dalloc(c, &c->flag, 1)) return bail(FR_ERR_ALLOC);
  if (hipMemcpy(c->perm, c->host.orient_perm.data(), c->host.orient_perm.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
    c->err = "upload failed";
    return bail(FR_ERR_DEVICE);
  }
  bool has_tet = false;
  for (auto& b : c->blocks) has_tet = has_tet || b.etype == FR_TET;
  if (has_tet) {
    const TetOps& T = c->host.tet;
    // flux point -> collocated solution point, then per solution point its flux points
    std::vector<int32_t> src(T.fp_src, T.fp_src + 60);
    src.resize(60 + 35 * 4, 0);
    for (int sg = 0; sg < 60; ++sg) {
      int32_t* row = &src[60 + 4 * T.fp_src[sg]];
      if (row[0] >= 3) { c->err = "a solution point collocated with more than 3 flux points"; return bail(FR_ERR_STATE); }
      row[1 + row[0]++] = sg;
    }
    // transposed, zero-padded divergence operator [Dh_0 Dh_1 Dh_2 L] of the matrix-core contraction
    std::vector<double> opT((size_t)TET_KP * TET_MP, 0.0);
    for (int k = 0; k < 105; ++k)
      for (int pt = 0; pt < 35; ++pt) opT[(size_t)k * TET_MP + pt] = T.Dh[k / 35][pt][k % 35];
    for (int sg = 0; sg < 60; ++sg)
      for (int pt = 0; pt < 35; ++pt) opT[(size_t)(TET_KA + sg) * TET_MP + pt] = T.lift[pt][sg];
    std::vector<char> bop(opT.size() * tsz);
    if (tsz == sizeof(float)) for (size_t i = 0; i < opT.size(); ++i) ((float*)bop.data())[i] = (float)opT[i];
    else std::memcpy(bop.data(), opT.data(), bop.size());
    // stacked, transposed gradient operator [[Dh_i, L diag(n~_i)]] (i = 0, 1, 2)
    std::vector<double> ogT((size_t)TGR_K * TGR_M, 0.0);
    for (int i = 0; i < 3; ++i)
      for (int pt = 0; pt < 35; ++pt) {
        for (int k = 0; k < 35; ++k) ogT[(size_t)k * TGR_M + TET_MP * i + pt] = T.Dh[i][pt][k];
        for (int sg = 0; sg < 60; ++sg)
          ogT[(size_t)(35 + sg) * TGR_M + TET_MP * i + pt] = T.lift[pt][sg] * T.nref[T.fp_face[sg]][i];
      }
    // Output-row order of the gradient product: rows {16 w + 4 g + q : g = 0..3} are the
    // ones the lanes of wave w visit together at step q of the common-flux loop, so points
    // are grouped by their number of flux points (3, 2, 1, 0) into such quadruples, and
    // the quadruples are dealt to the three waves so their loop trips balance.
    std::vector<int> slot_pt(TET_MP, -1);
    {
      std::vector<int> order(35);
      for (int z = 0; z < 35; ++z) order[z] = z;
      auto nfp_of = [&](int z) { return src[60 + 4 * z]; };
      std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return nfp_of(a) > nfp_of(b); });
      order.resize(TET_MP, -1);
      // 12 quadruples, costs = the largest flux-point count in each
      std::vector<int> cost(12, 0);
      for (int g = 0; g < 12; ++g)
        for (int j = 0; j < 4; ++j) if (order[4 * g + j] >= 0) cost[g] = std::max(cost[g], nfp_of(order[4 * g + j]));
      int load[3] = {0, 0, 0}, used[3] = {0, 0, 0};
      for (int g = 0; g < 12; ++g) {            // costs are non-increasing in g
        int wbest = -1;
        for (int w = 0; w < 3; ++w)
          if (used[w] < 4 && (wbest < 0 || load[w] < load[wbest])) wbest = w;
        const int q = used[wbest]++;
        load[wbest] += cost[g];
        for (int j = 0; j < 4; ++j) slot_pt[16 * wbest + 4 * j + q] = order[4 * g + j];
      }
    }
    std::vector<int> pt_slot(35, -1);
    for (int r = 0; r < TET_MP; ++r) if (slot_pt[r] >= 0) pt_slot[slot_pt[r]] = r;
    for (int r = 0; r < TET_MP; ++r) src.push_back(slot_pt[r]);
    // the same operator in the face-sparse row order of the FP32 / FP64 kernels (tgs_row):
    // direction i reads only the rows of faces 2 - i and 3, whose normals have an i component
    std::vector<double> ogS((size_t)TGS_K * TGR_M, 0.0);
    for (int i = 0; i < 3; ++i)
      for (int pt = 0; pt < 35; ++pt) {
        for (int k = 0; k < 35; ++k) ogS[(size_t)k * TGR_M + TET_MP * i + pt_slot[pt]] = T.Dh[i][pt][k];
        for (int sg = 0; sg < 60; ++sg) {
          const int f = T.fp_face[sg];
          if (f != sg / TET_NFPF || ((f != 2 - i && f != 3) && T.nref[f][i] != 0.0)) {
            c->err = "tetrahedral flux points not ordered by face, or a face normal off the expected axes";
            return bail(FR_ERR_STATE);
          }
          ogS[(size_t)(TGS_U + 16 * f + sg % TET_NFPF) * TGR_M + TET_MP * i + pt_slot[pt]] =
              T.lift[pt][sg] * T.nref[f][i];
        }
      }
    std::vector<char> bog(ogS.size() * tsz);
    if (tsz == sizeof(float)) for (size_t i = 0; i < ogS.size(); ++i) ((float*)bog.data())[i] = (float)ogS[i];
    else std::memcpy(bog.data(), ogS.data(), bog.size());
    if (p->precision == FR_FP32_BF16X3) {
      // [M][K] row-major (k contiguous), hi then lo, K padded to multiples of 16
      std::vector<uint16_t> dh((size_t)2 * TET_MP * TET_KP16, 0), gh((size_t)2 * TGR_M * TGR_K, 0);
      const size_t dlo = (size_t)TET_MP * TET_KP16, glo = (size_t)TGR_M * TGR_K;
      for (int m = 0; m < TET_MP; ++m) {
        for (int k = 0; k < 105; ++k) bf16_split_host(opT[(size_t)k * TET_MP + m], dh[(size_t)m * TET_KP16 + k],
                                                      dh[dlo + (size_t)m * TET_KP16 + k]);
        for (int s2 = 0; s2 < 60; ++s2)
          bf16_split_host(opT[(size_t)(TET_KA + s2) * TET_MP + m], dh[(size_t)m * TET_KP16 + TET_KA16 + s2],
                          dh[dlo + (size_t)m * TET_KP16 + TET_KA16 + s2]);
      }
      for (int i = 0; i < 3; ++i)
        for (int r = 0; r < TET_MP; ++r) {
          const int m = TET_MP * i + r, pt = slot_pt[r];
          if (pt < 0) continue;
          for (int k = 0; k < TGR_K; ++k)
            bf16_split_host(ogT[(size_t)k * TGR_M + TET_MP * i + pt], gh[(size_t)m * TGR_K + k],
                            gh[glo + (size_t)m * TGR_K + k]);
        }
      if (dalloc(c, (char**)&c->tet_opH, dh.size() * 2) || dalloc(c, (char**)&c->tet_ogH, gh.size() * 2) ||
          hipMemcpy(c->tet_opH, dh.data(), dh.size() * 2, hipMemcpyHostToDevice) != hipSuccess ||
          hipMemcpy(c->tet_ogH, gh.data(), gh.size() * 2, hipMemcpyHostToDevice) != hipSuccess) {
        c->err = "tet operator upload failed";
        return bail(FR_ERR_DEVICE);
      }
    }
    if (dalloc(c, (char**)&c->tet_opT, bop.size()) || dalloc(c, (char**)&c->tet_ogT, bog.size()) ||
        hipMemcpy(c->tet_opT, bop.data(), bop.size(), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(c->tet_ogT, bog.data(), bog.size(), hipMemcpyHostToDevice) != hipSuccess) {
      c->err = "tet operator upload failed";
      return bail(FR_ERR_DEVICE);
    }
    // per orientation and partner face: the partner's solution point of each flux point of
    // the face (bytes, behind the other tables); orientations of hexahedral faces unused
    {
      const int no = c->host.n_orient, st = c->host.perm_stride;
      std::vector<uint8_t> ps((size_t)no * 4 * 16, 0);
      for (int o = 0; o < no; ++o)
        for (int f = 0; f < 4; ++f)
          for (int q = 0; q < TET_NFPF && q < st; ++q) {
            const int pq = c->host.orient_perm[(size_t)o * st + q];
            if (pq >= 0 && pq < TET_NFPF) ps[((size_t)o * 4 + f) * 16 + q] = (uint8_t)T.fp_src[f * TET_NFPF + pq];
          }
      const size_t n0 = src.size();
      src.resize(n0 + ps.size() / 4);
      std::memcpy(&src[n0], ps.data(), ps.size());
    }
    if (dalloc(c, &c->tet_src, src.size())) return bail(FR_ERR_ALLOC);
    if (hipMemcpy(c->tet_src, src.data(), src.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
      c->err = "upload failed";
      return bail(FR_ERR_DEVICE);
    }
  }
  if (std::any_of(c->blocks.begin(), c->blocks.end(), [](const DevBlock& b) { return b.etype == FR_PYR; })) {
    const PyrOps& Y = c->host.pyr;
    // the general kernels' operators, then the matrix-core kernels' (zero-padded)
    const size_t pym0 = (size_t)PY_NSP * PY_NFP * 2 + 3 * PY_NSP * PY_NSP;
    std::vector<double> ops(pym0 + (size_t)PYM_KP * PYM_FM + 3 * PYM_KP * PYM_M + PYM_KL * PYM_M, 0.0);
    double* Im = ops.data() + pym0;
    double* Dm = Im + PYM_KP * PYM_FM;
    double* Lm = Dm + 3 * PYM_KP * PYM_M;
    for (int f = 0; f < 5; ++f) {
      // the flux tiles' layout and the sparsity of the normals that pyr_div_mma relies on
      const int flat = f == 0 ? 0 : (f % 2 ? 0 : 1);
      if (Y.face_off[f] != pym_off(f) || Y.face_off[f + 1] != pym_off(f + 1) || std::fabs(Y.nref[f][flat]) > 1e-14 ||
          (f == 0 && std::fabs(Y.nref[0][1]) > 1e-14)) {
        c->err = "pyramid faces not in the expected order";
        return bail(FR_ERR_STATE);
      }
    }
    for (int ft = 0; ft < PYM_FT; ++ft)
      for (int row = 0; row < 16; ++row) {
        const int fp = pym_fp(ft, row);
        if (fp < 0) continue;
        for (int j = 0; j < PY_NSP; ++j) Im[j * PYM_FM + 16 * ft + row] = Y.interp[fp][j];
        const int f = pym_face(ft), k = pym_krow0(f) + fp - pym_off(f);
        for (int pt = 0; pt < PY_NSP; ++pt) Lm[k * PYM_M + pt] = Y.lift[pt][fp];
      }
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < PY_NSP; ++j)
        for (int pt = 0; pt < PY_NSP; ++pt) Dm[(i * PYM_KP + j) * PYM_M + pt] = Y.D[i][pt][j];
    double* It = ops.data();
    double* Dt = It + PY_NSP * PY_NFP;
    double* Lt = Dt + 3 * PY_NSP * PY_NSP;
    for (int j = 0; j < PY_NSP; ++j)
      for (int fp = 0; fp < PY_NFP; ++fp) It[j * PY_NFP + fp] = Y.interp[fp][j];
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < PY_NSP; ++j)
        for (int pt = 0; pt < PY_NSP; ++pt) Dt[(i * PY_NSP + j) * PY_NSP + pt] = Y.D[i][pt][j];
    for (int fp = 0; fp < PY_NFP; ++fp)
      for (int pt = 0; pt < PY_NSP; ++pt) Lt[fp * PY_NSP + pt] = Y.lift[pt][fp];
    std::vector<char> bo(ops.size() * tsz);
    if (tsz == sizeof(float)) for (size_t i = 0; i < ops.size(); ++i) ((float*)bo.data())[i] = (float)ops[i];
    else std::memcpy(bo.data(), ops.data(), bo.size());
    if (dalloc(c, (char**)&c->pyr_ops, bo.size()) ||
        hipMemcpy(c->pyr_ops, bo.data(), bo.size(), hipMemcpyHostToDevice) != hipSuccess) {
      c->err = "pyramid operator upload failed";
      return bail(FR_ERR_DEVICE);
    }
  }
  *out = c;
  return FR_OK;
}
}  // namespace

fr_status fr_setup_mesh(const fr_params* p, int64_t n_vert, const double* xyz, const double* period,
                        int64_t n_elem, const int32_t* etype, const int64_t* enodes, void* stream,
                        fr_ctx* out) {
  return setup_impl(p, n_vert, xyz, period, n_elem, etype, enodes, 0, nullptr, stream, out);
}

fr_status fr_setup_mesh_curved(const fr_params* p, int32_t geo_order, int64_t n_vert, const double* xyz,
                               const double* period, int64_t n_elem, const int64_t* ho_nodes, void* stream,
                               fr_ctx* out) {
  if (!out) return fail(nullptr, FR_ERR_ARG, "out is NULL");
  *out = nullptr;
  if (!p || p->struct_size != sizeof(fr_params)) return fail(nullptr, FR_ERR_ARG, "fr_params missing or struct_size mismatch");
  if (!xyz || !period || !ho_nodes || n_vert <= 0 || n_elem <= 0) return fail(nullptr, FR_ERR_ARG, "empty mesh or NULL array");
  if (geo_order < 1 || geo_order > 4) return fail(nullptr, FR_ERR_UNSUPPORTED, "geometry order must be in 1..4");
  if (geo_order > p->order)
    return fail(nullptr, FR_ERR_UNSUPPORTED, "geometry order above the solution order (periodic faces would not be watertight)");
  const int nq = geo_order + 1, NQ = nq * nq * nq;
  for (int64_t i = 0; i < n_elem * NQ; ++i)
    if (ho_nodes[i] < 0 || ho_nodes[i] >= n_vert) return fail(nullptr, FR_ERR_ARG, "node index out of range");
  // the 8 corners in VTK order: tensor nodes with each index 0 or q
  static const int kc[8][3] = {{0, 0, 0}, {1, 0, 0}, {1, 1, 0}, {0, 1, 0}, {0, 0, 1}, {1, 0, 1}, {1, 1, 1}, {0, 1, 1}};
  std::vector<int64_t> corners((size_t)n_elem * 8);
  for (int64_t e = 0; e < n_elem; ++e)
    for (int c = 0; c < 8; ++c) {
      const int i = kc[c][0] * geo_order, j = kc[c][1] * geo_order, k = kc[c][2] * geo_order;
      corners[(size_t)e * 8 + c] = ho_nodes[e * NQ + i + nq * (j + nq * k)];
    }
  std::vector<int32_t> et((size_t)n_elem, FR_HEX);
  return setup_impl(p, n_vert, xyz, period, n_elem, et.data(), corners.data(), geo_order, ho_nodes, stream, out);
}

fr_status fr_setup_mesh_curved_tet(const fr_params* p, int32_t geo_order, int64_t n_vert, const double* xyz,
                                   const double* period, int64_t n_elem, const int64_t* ho_nodes, void* stream,
                                   fr_ctx* out) {
  if (!out) return fail(nullptr, FR_ERR_ARG, "out is NULL");
  *out = nullptr;
  if (!p || p->struct_size != sizeof(fr_params)) return fail(nullptr, FR_ERR_ARG, "fr_params missing or struct_size mismatch");
  if (!xyz || !period || !ho_nodes || n_vert <= 0 || n_elem <= 0) return fail(nullptr, FR_ERR_ARG, "empty mesh or NULL array");
  if (geo_order < 1 || geo_order > 4) return fail(nullptr, FR_ERR_UNSUPPORTED, "geometry order must be in 1..4");
  const int q = geo_order, NQ = (q + 1) * (q + 2) * (q + 3) / 6;
  for (int64_t i = 0; i < n_elem * NQ; ++i)
    if (ho_nodes[i] < 0 || ho_nodes[i] >= n_vert) return fail(nullptr, FR_ERR_ARG, "node index out of range");
  // node (i, j, k) has index k-outer, j, i-inner among i + j + k <= q; the corners in
  // reference order are the nodes (0,0,0), (q,0,0), (0,0,q), (0,q,0)
  auto node_id = [q](int i, int j, int k) {
    int id = 0;
    for (int kk = 0; kk < k; ++kk) id += (q + 1 - kk) * (q + 2 - kk) / 2;
    for (int jj = 0; jj < j; ++jj) id += q + 1 - k - jj;
    return id + i;
  };
  const int cid[4] = {node_id(0, 0, 0), node_id(q, 0, 0), node_id(0, 0, q), node_id(0, q, 0)};
  std::vector<int64_t> corners((size_t)n_elem * 8, -1);
  for (int64_t e = 0; e < n_elem; ++e)
    for (int c = 0; c < 4; ++c) corners[(size_t)e * 8 + c] = ho_nodes[e * NQ + cid[c]];
  std::vector<int32_t> et((size_t)n_elem, FR_TET);
  return setup_impl(p, n_vert, xyz, period, n_elem, et.data(), corners.data(), geo_order, ho_nodes, stream, out);
}

fr_status fr_layout(fr_ctx c, fr_layout_t* o) {
  if (!c || !o) return fail(c, FR_ERR_ARG, "NULL argument");
  std::memset(o, 0, sizeof(*o));
  o->n_types = (int32_t)c->blocks.size();
  for (size_t i = 0; i < c->blocks.size(); ++i) {
    const DevBlock& b = c->blocks[i];
    o->etype[i] = b.etype; o->n_elem[i] = b.n; o->e_pad[i] = b.E; o->n_sp[i] = b.nsp; o->n_fp[i] = b.nfp;
    o->canon_offset[i] = b.canon_off; o->native_offset[i] = b.native_off;
  }
  o->canon_len = c->canon_len;
  o->native_len = c->native_len;
  o->native_dtype = c->prm.precision == FR_FP64 ? FR_FP64 : FR_FP32;
  return FR_OK;
}

fr_status fr_sol_points(fr_ctx c, double* xyz) {
  if (!c || !xyz) return fail(c, FR_ERR_ARG, "NULL argument");
  size_t off = 0;
  for (auto& hb : c->host.blocks) {
    std::memcpy(xyz + off, hb.sol_xyz.data(), hb.sol_xyz.size() * sizeof(double));
    off += hb.sol_xyz.size();
  }
  return FR_OK;
}

}  // extern "C"

namespace {

// Every block of a canonical array to native values, or back.
template <typename T>
fr_status pack_blocks(fr_ctx c, const double* canon, T* native, RefVec ref) {
  for (auto& b : c->blocks) {
    const fr_status st = layout_block<T, true>(c, b, canon + b.canon_off, nullptr, nullptr, native + b.native_off, ref);
    if (st) return st;
  }
  HIP_TRY(c, hipGetLastError());
  return FR_OK;
}

template <typename T>
fr_status unpack_blocks(fr_ctx c, const T* native, double* canon, RefVec ref) {
  for (auto& b : c->blocks) {
    const fr_status st =
        layout_block<T, false>(c, b, nullptr, canon + b.canon_off, native + b.native_off, nullptr, ref);
    if (st) return st;
  }
  HIP_TRY(c, hipGetLastError());
  return FR_OK;
}

}  // namespace

extern "C" {

fr_status fr_pack(fr_ctx c, const double* canon, void* native) {
  if (!c || !canon || !native) return fail(c, FR_ERR_ARG, "NULL argument");
  if (c->prm.precision == FR_FP64) return pack_blocks<double>(c, canon, (double*)native, RefVec{});
  return pack_blocks<float>(c, canon, (float*)native, refvec(c->prm));
}

fr_status fr_unpack(fr_ctx c, const void* native, double* canon) {
  if (!c || !canon || !native) return fail(c, FR_ERR_ARG, "NULL argument");
  if (c->prm.precision == FR_FP64) return unpack_blocks<double>(c, (const double*)native, canon, RefVec{});
  return unpack_blocks<float>(c, (const float*)native, canon, refvec(c->prm));
}

fr_status fr_unpack_rhs(fr_ctx c, const void* r, double* canon) {
  if (!c || !canon || !r) return fail(c, FR_ERR_ARG, "NULL argument");
  if (c->prm.precision == FR_FP64) return unpack_blocks<double>(c, (const double*)r, canon, RefVec{});
  return unpack_blocks<float>(c, (const float*)r, canon, RefVec{});
}

fr_status fr_pack64(fr_ctx c, const double* canon, double* native) {
  if (!c || !canon || !native) return fail(c, FR_ERR_ARG, "NULL argument");
  return pack_blocks<double>(c, canon, native, RefVec{});
}

fr_status fr_unpack64(fr_ctx c, const double* native, double* canon) {
  if (!c || !canon || !native) return fail(c, FR_ERR_ARG, "NULL argument");
  return unpack_blocks<double>(c, native, canon, RefVec{});
}

fr_status fr_rhs(fr_ctx c, const void* u, void* r) {
  if (!c || !u || !r) return fail(c, FR_ERR_ARG, "NULL argument");
  if (u == r) return fail(c, FR_ERR_ARG, "u and r must not alias");
  return rhs_native(c, u, r);
}

}  // extern "C"

namespace {
// RK workspace.  Padding lanes of the increments are never written by the RHS and start at zero.
// What either integrator needs of the first call on is allocated by it whatever the filter
// (a later call with another one then allocates nothing of it), the embedded pair's own apart.
fr_status rk_alloc(fr_ctx c, bool pair) {
  const int64_t n = c->native_len;
  const bool f32 = c->prm.precision != FR_FP64;
  auto get = [&](void** p, size_t bytes) -> fr_status {
    if (*p) return FR_OK;
    if (dalloc(c, (char**)p, bytes)) return FR_ERR_ALLOC;
    HIP_TRY(c, hipMemsetAsync(*p, 0, bytes, c->stream));
    return FR_OK;
  };
  fr_status st;
  if ((st = get(&c->rk_stage, n * native_size(c))) || (st = get(&c->rk_k, n * native_size(c)))) return st;
  if (f32) return get(&c->rk_kk, 3 * n * sizeof(float));
  if ((st = get((void**)&c->rk_acc, n * sizeof(double)))) return st;
  return pair ? get(&c->rk_kk, 2 * n * sizeof(double)) : FR_OK;
}

// RK3(2)4[2R+]C (Kennedy, Carpenter & Lewis 2000): subdiagonal, weights, embedded weights.
constexpr double kLsA[3][2] = {{11847461282814.0, 36547543011857.0}, {3943225443063.0, 7078155732230.0},
                               {-346793006927.0, 4029903576067.0}};
constexpr double kLsB[4][2] = {{1017324711453.0, 9774461848756.0}, {8237718856693.0, 13685301971492.0},
                               {57731312506979.0, 19404895981398.0}, {-101169746363290.0, 37734290219643.0}};
constexpr double kLsBh[4][2] = {{15763415370699.0, 46270243929542.0}, {514528521746.0, 5659431552419.0},
                                {27030193851939.0, 9429696342944.0}, {-69544964788955.0, 30262026368149.0}};
constexpr int kNormGrid = 1024;
}  // namespace

extern "C" {

void fr_default_adaptive_params(fr_adaptive_params* p) {
  if (!p) return;
  p->atol = 1e-6;
  p->rtol = 1e-6;
  p->safety = 0.9;
  p->fac_min = 0.3;
  p->fac_max = 2.5;
  p->max_attempts = 100000;
  p->reserved = 0;
}

fr_status fr_rk_adaptive(fr_ctx c, void* u_, double t_end, double dt0, const fr_adaptive_params* ap,
                         fr_adaptive_stats* stats) {
  if (!c || !u_ || !ap) return fail(c, FR_ERR_ARG, "NULL argument");
  if (!(t_end > 0) || !std::isfinite(t_end) || !(dt0 > 0) || !std::isfinite(dt0))
    return fail(c, FR_ERR_ARG, "t_end and dt0 must be positive and finite");
  if (!(ap->atol > 0) || !(ap->rtol >= 0) || !(ap->safety > 0) || !(ap->safety <= 1) || !(ap->fac_min > 0) ||
      !(ap->fac_min <= 1) || !(ap->fac_max >= 1) || !std::isfinite(ap->fac_max) || ap->max_attempts < 1)
    return fail(c, FR_ERR_ARG, "adaptive parameters out of range");
  fr_status st;
  if ((st = rk_alloc(c, true))) return st;
  const int64_t n = c->native_len;
  if (!c->rk_part && dalloc(c, &c->rk_part, (int64_t)kNormGrid * (int64_t)c->blocks.size())) return FR_ERR_ALLOC;
  if (c->prm.precision != FR_FP64 && !c->rk_x0 && dalloc(c, &c->rk_x0, n)) return FR_ERR_ALLOC;
  double* X = (double*)u_;
  const bool f32 = c->prm.precision != FR_FP64;
  const RefVec ref = refvec(c->prm);
  int64_t count = 0;
  for (auto& b : c->blocks) count += b.n * b.nsp * 5;
  std::vector<double> part(c->blocks.size() * kNormGrid);
  // u_n for a rejected step: in FP64 the stage state's buffer, which the last stage has read
  double* X0 = f32 ? c->rk_x0 : (double*)c->rk_stage;
  // one stage update on every block
  auto stage_t = [&](int i, double h, auto kt) {
    using KT = decltype(kt);
    for (size_t bi = 0; bi < c->blocks.size(); ++bi) {
      const DevBlock& b = c->blocks[bi];
      const int64_t o = b.native_off;
      LsK<KT> A;
      for (int j = 0; j < 4; ++j) {
        A.k[j] = (const KT*)rk_inc(c, b, j);
        A.xb[j] = h * (kLsB[j][0] / kLsB[j][1]);
        A.ed[j] = h * (kLsB[j][0] / kLsB[j][1] - kLsBh[j][0] / kLsBh[j][1]);
      }
      A.ya = i < 3 ? h * (kLsA[i][0] / kLsA[i][1]) : 0.0;
      const int rows = b.nsp * 5, nt = b.E >= 512 ? 256 : 64;
      const dim3 grid((unsigned)((b.E + nt - 1) / nt), (unsigned)rows);
      KT* Y = (KT*)c->rk_stage + o;
      if (i == 0) k_lsrk_stage<KT, 0><<<grid, nt, 0, c->stream>>>(X + o, A, Y, b.E, b.n, rows, ref);
      else if (i == 1) k_lsrk_stage<KT, 1><<<grid, nt, 0, c->stream>>>(X + o, A, Y, b.E, b.n, rows, ref);
      else if (i == 2) k_lsrk_stage<KT, 2><<<grid, nt, 0, c->stream>>>(X + o, A, Y, b.E, b.n, rows, ref);
      else
        k_lsrk_last<KT><<<kNormGrid, 256, 0, c->stream>>>(X + o, A, X0 + o, rows * b.E, b.E, b.n, ap->atol, ap->rtol,
                                                          c->rk_part + bi * kNormGrid);
    }
  };
  auto stage = [&](int i, double h) {
    if (f32) stage_t(i, h, float());
    else stage_t(i, h, double());
  };
  fr_adaptive_stats s{};
  double t = 0.0, dt = dt0, nrm = 0.0;
  while (t < t_end && s.accepted + s.rejected < ap->max_attempts) {
    const bool last = dt >= t_end - t;
    const double h = last ? t_end - t : dt;
    for (int i = 0; i < 4; ++i) {
      void* in = c->rk_stage;
      if (i == 0) {
        if (f32) {
          for (auto& b : c->blocks) {
            const int64_t nb = (int64_t)b.nsp * 5 * b.E, o = b.native_off;
            k_to_dev<<<grid_for(nb, 256), 256, 0, c->stream>>>(X + o, (float*)c->rk_stage + o, nb, b.E, ref);
          }
        } else {
          in = X;
        }
      }
      void* ks[kMaxBlocks] = {};
      for (size_t bi = 0; bi < c->blocks.size(); ++bi) ks[bi] = rk_inc(c, c->blocks[bi], i);
      if ((st = rhs_blocks(c, in, ks))) return st;
      stage(i, h);
    }
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipMemcpyAsync(part.data(), c->rk_part, part.size() * sizeof(double), hipMemcpyDeviceToHost,
                              c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    double sum = 0.0;
    for (double v : part) sum += v;
    nrm = std::sqrt(sum / (double)count);
    s.n_rhs += 4;
    if (nrm <= 1.0) {
      t = last ? t_end : t + h;
      ++s.accepted;
    } else {
      HIP_TRY(c, hipMemcpyAsync(X, X0, n * sizeof(double), hipMemcpyDeviceToDevice, c->stream));
      ++s.rejected;
    }
    double fac;
    if (!std::isfinite(nrm)) fac = ap->fac_min;
    else if (nrm == 0.0) fac = ap->fac_max;
    else fac = std::min(ap->fac_max, std::max(ap->fac_min, ap->safety * std::pow(nrm, -1.0 / 3.0)));
    dt = h * fac;
  }
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  s.t = t;
  s.dt_next = dt;
  s.last_norm = nrm;
  if (stats) *stats = s;
  return FR_OK;
}

fr_status fr_rk_step(fr_ctx c, void* u_, double dt, int32_t n_steps, int32_t filter_mode) {
  if (!c || !u_) return fail(c, FR_ERR_ARG, "NULL argument");
  if (n_steps < 0 || !std::isfinite(dt)) return fail(c, FR_ERR_ARG, "n_steps or dt");
  if (filter_mode < -1 || filter_mode > 1) return fail(c, FR_ERR_ARG, "filter_mode must be -1, 0 or 1");
  if (filter_mode == 1 && !c->mlp_ready) return fail(c, FR_ERR_STATE, "MLP weights not set");
  if (filter_mode >= 0) {
    fr_status fs = filter_alloc(c);
    if (fs) return fs;
  }
  double* u = (double*)u_;
  const int64_t n = c->native_len;
  const bool f32 = c->prm.precision != FR_FP64;
  fr_status st;
  if ((st = rk_alloc(c, false))) return st;
  const int g = grid_for(n, 256);
  const double b1 = dt / 6.0, b2 = dt / 3.0, c2 = dt / 2.0;
  int pk;
  if (!f32) {
    double *K = (double*)c->rk_k, *S = (double*)c->rk_stage;
    const bool filt = filter_mode >= 0;
    if (filt && !c->collecting) {
      // each stage update runs inside the filter's detection pass (the stage state is
      // checked as it is formed instead of being read back)
      for (int s = 0; s < n_steps; ++s) {
        if ((st = compute_smin(c, u))) return st;
        for (int stage = 0; stage < 4; ++stage) {
          if ((st = rhs_native(c, stage == 0 ? u : S, K))) return st;
          StageFuse fz;
          fz.stage = stage;
          fz.b = stage == 0 || stage == 3 ? b1 : b2;
          fz.c = stage == 2 ? dt : c2;
          fz.u = u;
          fz.s64 = stage < 3 ? S : nullptr;
          if ((st = apply_filter(c, stage < 3 ? S : u, filter_mode, nullptr, &fz))) return st;
        }
      }
      HIP_TRY(c, hipGetLastError());
      return FR_OK;
    }
    for (int s = 0; s < n_steps; ++s) {
      // entropy bound of this step from u_n; every later stage state and u_{n+1} is filtered
      if (filt && (st = compute_smin(c, u))) return st;
      if ((st = rhs_native(c, u, K))) return st;
      pk = c->prof_begin("rk4_update");
      k_rk_first<double><<<g, 256, 0, c->stream>>>(u, K, c->rk_acc, S, n, b1, c2);
      c->prof_end(pk);
      if (filt && (st = apply_filter(c, S, filter_mode))) return st;
      if ((st = rhs_native(c, S, K))) return st;
      pk = c->prof_begin("rk4_update");
      k_rk_mid<double><<<g, 256, 0, c->stream>>>(u, K, c->rk_acc, S, n, b2, c2);
      c->prof_end(pk);
      if (filt && (st = apply_filter(c, S, filter_mode))) return st;
      if ((st = rhs_native(c, S, K))) return st;
      pk = c->prof_begin("rk4_update");
      k_rk_mid<double><<<g, 256, 0, c->stream>>>(u, K, c->rk_acc, S, n, b2, dt);
      c->prof_end(pk);
      if (filt && (st = apply_filter(c, S, filter_mode))) return st;
      if ((st = rhs_native(c, S, K))) return st;
      pk = c->prof_begin("rk4_update");
      k_rk_last<double><<<g, 256, 0, c->stream>>>(u, K, c->rk_acc, n, b1);
      c->prof_end(pk);
      if (filt && (st = apply_filter(c, u, filter_mode))) return st;
    }
  } else {
    float* S = (float*)c->rk_stage;
    const RefVec ref = refvec(c->prm);
    // the right-hand side of a stage into its kept increment; the fused hexahedral filter, which
    // keeps an accumulator instead, reads the stage's own alone
    auto stage_rhs = [&](int stage, bool fused) {
      void* ks[kMaxBlocks] = {};
      for (size_t bi = 0; bi < c->blocks.size(); ++bi)
        ks[bi] = rk_inc(c, c->blocks[bi], fused && c->blocks[bi].etype == FR_HEX ? 3 : stage);
      return rhs_blocks(c, S, ks);
    };
    // the FP32 deviation of u_n; later steps get it from the previous step's last update
    for (auto& b : c->blocks) {
      const int64_t nb = (int64_t)b.nsp * 5 * b.E;
      k_to_dev<<<grid_for(nb, 256), 256, 0, c->stream>>>(u + b.native_off, S + b.native_off, nb, b.E, ref);
    }
    if (filter_mode >= 0) {
      // filtered: every stage state is formed in FP64 (for the filter and its FP64
      // checks) together with the FP32 deviation the kernels read
      if (!c->rk_s64 && dalloc(c, &c->rk_s64, n)) return FR_ERR_ALLOC;
      double* S64 = c->rk_s64;
      if (!c->collecting) {
        // each stage update runs inside the filter's detection pass: the FP64 stage state
        // is formed in registers and checked there, its FP32 deviation written for the
        // next right-hand side, and only the candidates' FP64 states written for the search
        for (int s = 0; s < n_steps; ++s) {
          if ((st = compute_smin(c, u))) return st;
          for (int stage = 0; stage < 4; ++stage) {
            if ((st = stage_rhs(stage, true))) return st;
            StageFuse fz;
            fz.stage = stage;
            fz.b = stage == 0 || stage == 3 ? b1 : b2;
            fz.c = stage == 2 ? dt : c2;
            fz.k32 = true;
            fz.b1 = b1;
            fz.b2 = b2;
            fz.u = u;
            fz.s32 = S;
            fz.cand64 = stage < 3 ? S64 : nullptr;
            if ((st = apply_filter(c, stage < 3 ? S64 : u, filter_mode, S, &fz))) return st;
          }
        }
        HIP_TRY(c, hipGetLastError());
        return FR_OK;
      }
    }
    // unfiltered, or collecting training data (the filter then works on whole FP64 stage states
    // and rewrites the FP32 deviation of every element it changes)
    for (int s = 0; s < n_steps; ++s) {
      if (filter_mode >= 0 && (st = compute_smin(c, u))) return st;
      for (int stage = 0; stage < 4; ++stage) {
        if ((st = stage_rhs(stage, false))) return st;
        pk = c->prof_begin("rk4_update_f32");
        for (auto& b : c->blocks) {
          const int64_t o = b.native_off;
          const int rows = b.nsp * 5, nt = b.E >= 512 ? 256 : 32;
          const dim3 grid((unsigned)((b.E / 2 + nt - 1) / nt), (unsigned)rows);
          auto inc = [&](int s) { return (const float*)rk_inc(c, b, s); };
          const Rk32 A{u + o, inc(0), inc(1), inc(2), inc(stage), S + o, filter_mode >= 0 ? c->rk_s64 + o : nullptr,
                       b1, b2, stage == 2 ? dt : c2};
          if (stage < 3) k_rk32<false><<<grid, nt, 0, c->stream>>>(A, b.E, b.n, rows, ref);
          else k_rk32<true><<<grid, nt, 0, c->stream>>>(A, b.E, b.n, rows, ref);
        }
        c->prof_end(pk);
        if (filter_mode >= 0 && (st = apply_filter(c, stage < 3 ? c->rk_s64 : u, filter_mode, S))) return st;
      }
    }
  }
  HIP_TRY(c, hipGetLastError());
  return FR_OK;
}

fr_status fr_check(fr_ctx c, const void* u) {
  if (!c || !u) return fail(c, FR_ERR_ARG, "NULL argument");
  HIP_TRY(c, hipMemsetAsync(c->flag, 0, sizeof(int), c->stream));
  for (auto& b : c->blocks) {
    k_check<<<grid_for(b.n * b.nsp, 256), 256, 0, c->stream>>>((const double*)u + b.native_off, b.n, b.E, b.nsp,
                                                              c->prm.gamma - 1.0, c->flag);
  }
  int h = 0;
  HIP_TRY(c, hipMemcpyAsync(&h, c->flag, sizeof(int), hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return h ? fail(c, FR_ERR_NONFINITE, "non-finite value or non-positive density/pressure") : FR_OK;
}

fr_status fr_profile(fr_ctx c, int32_t enable) {
  if (!c) return fail(c, FR_ERR_ARG, "NULL context");
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  if (enable) c->prof_clear();
  c->prof = enable != 0;
  return FR_OK;
}

fr_status fr_profile_read(fr_ctx c, fr_kernel_time* out, int32_t cap, int32_t* n) {
  if (!c || !n || (cap > 0 && !out)) return fail(c, FR_ERR_ARG, "NULL argument");
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  std::vector<fr_kernel_time> acc(c->prof_names.size());
  for (size_t i = 0; i < acc.size(); ++i) {
    std::memset(&acc[i], 0, sizeof(fr_kernel_time));
    std::strncpy(acc[i].name, c->prof_names[i].c_str(), sizeof(acc[i].name) - 1);
  }
  for (auto& e : c->prof_events) {
    float ms = 0;
    HIP_TRY(c, hipEventElapsedTime(&ms, e.a, e.b));
    acc[e.id].launches += 1;
    acc[e.id].total_ms += ms;
  }
  *n = (int32_t)acc.size();
  for (int32_t i = 0; i < cap && i < (int32_t)acc.size(); ++i) out[i] = acc[i];
  return FR_OK;
}

fr_status fr_sync(fr_ctx c) {
  if (!c) return fail(c, FR_ERR_ARG, "NULL context");
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return FR_OK;
}

fr_status fr_filter(fr_ctx c, void* u_, const void* uprev_, int32_t mode, int32_t* k_dev, fr_filter_stats* stats) {
  if (!c || !u_ || !uprev_) return fail(c, FR_ERR_ARG, "NULL argument");
  if (mode != 0 && mode != 1) return fail(c, FR_ERR_ARG, "mode must be 0 (plain) or 1 (MLP warm start)");
  if (mode == 1 && !c->mlp_ready) return fail(c, FR_ERR_STATE, "MLP weights not set");
  fr_status st;
  if ((st = filter_alloc(c))) return st;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (stats) {
    HIP_TRY(c, hipEventCreate(&e0));
    HIP_TRY(c, hipEventCreate(&e1));
    HIP_TRY(c, hipEventRecord(e0, c->stream));
  }
  if ((st = compute_smin(c, (const double*)uprev_))) return st;
  if ((st = apply_filter(c, (double*)u_, mode))) return st;
  if (k_dev)
    k_elem_to_canon<<<grid_for(c->n_elem_total, 256), 256, 0, c->stream>>>(c->f_k, c->g_npos, c->n_elem_total, k_dev);
  if (stats) {
    HIP_TRY(c, hipEventRecord(e1, c->stream));
    std::vector<int32_t> k(c->n_elem_total), ev(c->n_elem_total);
    HIP_TRY(c, hipMemcpyAsync(k.data(), c->f_k, k.size() * 4, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipMemcpyAsync(ev.data(), c->f_evals, ev.size() * 4, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    float ms = 0;
    HIP_TRY(c, hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    std::memset(stats, 0, sizeof(*stats));
    for (size_t i = 0; i < k.size(); ++i) {
      if (k[i] != 0) { stats->n_troubled++; stats->n_evals += ev[i]; }
      if (k[i] < 0) stats->n_fallback++;
    }
    stats->seconds = ms * 1e-3;
    for (auto& b : c->blocks) {
      int32_t m = 0;
      HIP_TRY(c, hipMemcpy(&m, b.f_cnt + c->f_slot, 4, hipMemcpyDeviceToHost));
      stats->n_candidates += m;
    }
  }
  return FR_OK;
}

fr_status fr_mlp_set_weights(fr_ctx c, const float* w, const float* xm, const float* xs) {
  if (!c || !w || !xm || !xs) return fail(c, FR_ERR_ARG, "NULL argument");
  for (int i = 0; i < MLP_IN; ++i)
    if (!(xs[i] > 0)) return fail(c, FR_ERR_ARG, "x_std must be positive");
  fr_status st;
  if ((st = mlp_alloc(c, 1))) return st;
  std::vector<float> sc(2 * MLP_IN);
  for (int i = 0; i < MLP_IN; ++i) { sc[i] = xm[i]; sc[MLP_IN + i] = xs[i]; }
  HIP_TRY(c, hipMemcpyAsync(c->m_w, w, MLP_NP * sizeof(float), hipMemcpyHostToDevice, c->stream));
  HIP_TRY(c, hipMemcpyAsync(c->m_scale, sc.data(), sc.size() * sizeof(float), hipMemcpyHostToDevice, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  c->mlp_ready = true;
  return FR_OK;
}

fr_status fr_mlp_get_weights(fr_ctx c, float* w) {
  if (!c || !w) return fail(c, FR_ERR_ARG, "NULL argument");
  if (!c->mlp_ready) return fail(c, FR_ERR_STATE, "MLP weights not set");
  HIP_TRY(c, hipMemcpyAsync(w, c->m_w, MLP_NP * sizeof(float), hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return FR_OK;
}

fr_status fr_mlp_features(fr_ctx c, const void* u_, const void* uprev_, float* x, int32_t* elem, int32_t* kout,
                          int64_t cap, int64_t* n) {
  if (!c || !u_ || !uprev_ || !n || (cap > 0 && !x)) return fail(c, FR_ERR_ARG, "NULL argument");
  fr_status st;
  if ((st = filter_alloc(c))) return st;
  if (!c->f_copy && dalloc(c, &c->f_copy, c->native_len)) return FR_ERR_ALLOC;
  if ((st = compute_smin(c, (const double*)uprev_))) return st;
  if ((st = candidate_features(c, (const double*)u_))) return st;
  // training targets: the plain search on a copy of the state
  HIP_TRY(c, hipMemcpyAsync(c->f_copy, u_, c->native_len * sizeof(double), hipMemcpyDeviceToDevice, c->stream));
  if ((st = apply_filter(c, c->f_copy, 0))) return st;
  std::vector<int32_t> flag(c->n_elem_total);
  HIP_TRY(c, hipMemcpyAsync(flag.data(), c->f_flag, flag.size() * 4, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  // rows in canonical element order
  std::vector<std::pair<int32_t, int32_t>> sel;
  for (size_t i = 0; i < flag.size(); ++i) if (flag[i]) sel.push_back({c->h_cpos[i], (int32_t)i});
  std::sort(sel.begin(), sel.end());
  std::vector<int32_t> idx(sel.size()), cid(sel.size());
  for (size_t i = 0; i < sel.size(); ++i) { cid[i] = sel[i].first; idx[i] = sel[i].second; }
  *n = (int64_t)idx.size();
  const int64_t m = std::min<int64_t>(cap, *n);
  if (m > 0) {
    int32_t* didx = nullptr;
    if (dalloc(c, &didx, m)) return FR_ERR_ALLOC;
    HIP_TRY(c, hipMemcpyAsync(didx, idx.data(), m * 4, hipMemcpyHostToDevice, c->stream));
    k_gather_features<<<(unsigned)((m + 255) / 256), 256, 0, c->stream>>>(c->f_feat, c->f_k, didx, m, x, nullptr,
                                                                          kout);
    if (elem) HIP_TRY(c, hipMemcpyAsync(elem, cid.data(), m * 4, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    (void)hipFree(didx);
  }
  return FR_OK;
}

fr_status fr_mlp_collect(fr_ctx c, void* u, double dt, int32_t n_steps, float* x, int32_t* k, int64_t cap,
                         int64_t* n) {
  if (!c || !u || !n || cap < 0 || (cap > 0 && (!x || !k))) return fail(c, FR_ERR_ARG, "bad argument");
  fr_status st;
  if ((st = filter_alloc(c))) return st;
  if (!c->f_copy && dalloc(c, &c->f_copy, c->native_len)) return FR_ERR_ALLOC;
  c->collecting = true;
  c->col_x = x;
  c->col_k = k;
  c->col_cap = cap;
  c->col_n = 0;
  c->col_seen = 0;
  st = fr_rk_step(c, u, dt, n_steps, 0);
  c->collecting = false;
  *n = c->col_n;
  return st;
}

fr_status fr_mlp_forward(fr_ctx c, const float* x, int64_t n, float* y) {
  if (!c || (n > 0 && (!x || !y)) || n < 0) return fail(c, FR_ERR_ARG, "bad argument");
  if (!c->mlp_ready) return fail(c, FR_ERR_STATE, "MLP weights not set");
  if (n == 0) return FR_OK;
  mlp_forward<<<(unsigned)((n + 255) / 256), 256, 0, c->stream>>>(c->m_w, c->m_scale, x, nullptr, n, 0, y);
  HIP_TRY(c, hipGetLastError());
  return FR_OK;
}

fr_status fr_mlp_grad(fr_ctx c, const float* x, const float* y, int64_t n, float* grad, float* loss) {
  if (!c || !x || !y || !grad || !loss || n <= 0 || n > (1 << 20)) return fail(c, FR_ERR_ARG, "bad argument");
  if (!c->mlp_ready) return fail(c, FR_ERR_STATE, "MLP weights not set");
  fr_status st;
  if ((st = mlp_alloc(c, (int)n))) return st;
  mlp_fwd_bwd<<<(unsigned)((n + MLP_FB_WAVES - 1) / MLP_FB_WAVES), 64 * MLP_FB_WAVES, 0, c->stream>>>(
      c->m_w, c->m_scale, x, y, nullptr, (int)n, c->m_scratch, c->m_sqerr);
  mlp_grad_reduce<false><<<MLP_NP / MLP_GR_P + 1, MLP_GR_NT, 0, c->stream>>>(c->m_scratch, (int)n, c->m_sqerr, grad,
                                                                            loss, AdamArgs{});
  HIP_TRY(c, hipGetLastError());
  return FR_OK;
}

fr_status fr_mlp_grad_static(fr_ctx c, const float* x, const float* y, int64_t n, float* grad, float* loss) {
  if (!c || !x || !y || !grad || !loss) return fail(c, FR_ERR_ARG, "NULL argument");
  if (n <= 0 || n > FR_MLP_STATIC_MAX_BATCH)
    return fail(c, FR_ERR_ARG, "batch size must be in 1..FR_MLP_STATIC_MAX_BATCH (4096)");
  if (!c->mlp_ready) return fail(c, FR_ERR_STATE, "MLP weights not set");
  if (!c->static_scratch) return fail(c, FR_ERR_DEVICE, "address of the static scratch array not available");
  float* S = c->static_scratch;
  float* sq = S + (int64_t)FR_MLP_STATIC_MAX_BATCH * MLP_SS;
  mlp_fwd_bwd<<<(unsigned)((n + MLP_FB_WAVES - 1) / MLP_FB_WAVES), 64 * MLP_FB_WAVES, 0, c->stream>>>(
      c->m_w, c->m_scale, x, y, nullptr, (int)n, S, sq);
  mlp_grad_reduce<false><<<MLP_NP / MLP_GR_P + 1, MLP_GR_NT, 0, c->stream>>>(S, (int)n, sq, grad, loss, AdamArgs{});
  HIP_TRY(c, hipGetLastError());
  return FR_OK;
}

fr_status fr_mlp_train(fr_ctx c, const float* x, const float* y, int64_t n, const int32_t* perm, int32_t n_steps,
                       int32_t batch, float lr, float b1, float b2, float eps, float* loss_hist) {
  if (!c || !x || !y || !perm || n <= 0 || n_steps < 0 || batch <= 0 || batch > (1 << 16))
    return fail(c, FR_ERR_ARG, "bad argument");
  if (!c->mlp_ready) return fail(c, FR_ERR_STATE, "MLP weights not set");
  fr_status st;
  if ((st = mlp_alloc(c, batch))) return st;
  HIP_TRY(c, hipMemsetAsync(c->m_m, 0, MLP_NP * sizeof(float), c->stream));
  HIP_TRY(c, hipMemsetAsync(c->m_v, 0, MLP_NP * sizeof(float), c->stream));
  for (int t = 1; t <= n_steps; ++t) {
    mlp_fwd_bwd<<<(unsigned)((batch + MLP_FB_WAVES - 1) / MLP_FB_WAVES), 64 * MLP_FB_WAVES, 0, c->stream>>>(
        c->m_w, c->m_scale, x, y, perm + (int64_t)(t - 1) * batch, batch, c->m_scratch, c->m_sqerr);
    const AdamArgs A{c->m_w, c->m_m, c->m_v, lr, b1, b2, eps, 1.0f - std::pow(b1, (float)t), 1.0f - std::pow(b2, (float)t)};
    mlp_grad_reduce<true><<<MLP_NP / MLP_GR_P + 1, MLP_GR_NT, 0, c->stream>>>(
        c->m_scratch, batch, c->m_sqerr, nullptr, loss_hist ? loss_hist + (t - 1) : c->m_loss, A);
  }
  HIP_TRY(c, hipGetLastError());
  return FR_OK;
}

}  // extern "C"
