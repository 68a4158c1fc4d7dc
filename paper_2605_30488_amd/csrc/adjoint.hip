// Hand-written adjoint of E_global (eq. 5) with the matches held fixed: gradients with respect to the
// canonical pointmaps, the confidences and a left tangent per pose, recomputing every edge's forward pass
// instead of storing Jacobians.
//
// With r_c = sqrt(q) e_c / sigma_c, q = sqrt(C_i C_j) and rho'(r) = w r (Sec. III-A):
//   gamma_c = dE/de_c = w_c q e_c / sigma_c^2,
//   dE/dx = P gamma_ray / d + gamma_range psi          (x = T_ij X_j, P = I - psi psi^T),
//   dE/dX_j[n] = (s_ij R_ij)^T dE/dx,  dE/dX_i[m] = -(P_i gamma_ray / d_i + gamma_range psi_i),
//   dE/dC = sum_c w_c r_c^2 / (4 C) for both endpoint confidences (r_c scales with (C_i C_j)^(1/4)),
//   dE/dtau_j = Ad^T [dE/dx; x x dE/dx; x . dE/dx] summed over the edge,  dE/dtau_i = -(the same)
//   (the chain of eq. 6 and the -/+Ad endpoint maps; equal to the Gauss-Newton gradient g).
// Two passes: the query side of every pixel is gathered over the edges that end in its keyframe and
// stored once (no atomics, which also clears the outputs); the gathered side then adds its terms with
// float atomics, since several matches of one edge can land on one pixel of i and a keyframe is the
// gathered side of several edges.
#include "common.hpp"
#include "internal.hpp"
#include "sim3.hpp"

namespace ds3 {

constexpr int kAdjThreads = 256;
constexpr int kAdjWaves = kAdjThreads / kWave;  // per-edge partials are written per wave (no block barrier)
constexpr int kAdjPPT = 2;  // 58 VGPRs, 8 waves per SIMD in the gather (4, at 99 VGPRs, was 15% slower; 1: the wave sums dominate)

// Forward pass and cotangents of one match (n of j, m of i), scaled by dcost. Returns false for the
// pixels the cost skips (holes, zero ranges, bad confidences, non-finite values).
struct AdjPix {
  float x[3];    // T_ij X_j[n]
  float gx[3];   // dE/dx
  float gam[4];  // dE/de
  float dc;      // sum_c w_c r_c^2
  float rho;     // Huber cost of the four components (not scaled by dcost)
};

__device__ inline bool adj_pixel(const float4 Xj, const float4 Xi, const float* M, const GnConst& k, float dcost,
                                 AdjPix& o) {
  const float x0 = fmaf(M[0], Xj.x, fmaf(M[1], Xj.y, fmaf(M[2], Xj.z, M[9])));
  const float x1 = fmaf(M[3], Xj.x, fmaf(M[4], Xj.y, fmaf(M[5], Xj.z, M[10])));
  const float x2 = fmaf(M[6], Xj.x, fmaf(M[7], Xj.y, fmaf(M[8], Xj.z, M[11])));
  const float d2 = fmaf(x0, x0, fmaf(x1, x1, x2 * x2));
  const float di2 = fmaf(Xi.x, Xi.x, fmaf(Xi.y, Xi.y, Xi.z * Xi.z));
  const float dj2 = fmaf(Xj.x, Xj.x, fmaf(Xj.y, Xj.y, Xj.z * Xj.z));
  const float cc = Xi.w * Xj.w;
  const float mn = fminf(fminf(d2, di2), dj2);
  const float sum = (d2 + di2) + (dj2 + cc);
  if (!(mn > 1e-18f) || !(cc >= 0.0f) || !(sum < __builtin_huge_valf())) return false;
  const float rd = rsqrtf(d2), rdi = rsqrtf(di2);
  const float d = d2 * rd, di = di2 * rdi;
  const float p[3] = {x0 * rd, x1 * rd, x2 * rd};
  const float e4[4] = {p[0] - Xi.x * rdi, p[1] - Xi.y * rdi, p[2] - Xi.z * rdi, d - di};
  const float sq = __builtin_amdgcn_sqrtf(__builtin_amdgcn_sqrtf(cc));
  const float isg[4] = {k.inv_sr, k.inv_sr, k.inv_sr, k.inv_sd};
  float dc = 0.0f, rho = 0.0f;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float r = sq * e4[c] * isg[c];
    const float a = fabsf(r);
    const float w = fminf(1.0f, k.kappa * __builtin_amdgcn_rcpf(a));
    o.gam[c] = w * r * sq * isg[c] * dcost;
    dc = fmaf(w * r, r, dc);
    const float t = w * a;  // rho = t (|r| - t/2)
    rho = fmaf(t, fmaf(-0.5f, t, a), rho);
  }
  o.rho = rho;
  o.dc = dc * dcost;
  const float pg = p[0] * o.gam[0] + p[1] * o.gam[1] + p[2] * o.gam[2];
#pragma unroll
  for (int a = 0; a < 3; ++a) o.gx[a] = (o.gam[a] - p[a] * pg) * rd + o.gam[3] * p[a];
  o.x[0] = x0;
  o.x[1] = x1;
  o.x[2] = x2;
  return true;
}

// The gathered side of one match alone: dE/dX_i[m] into g and sum_c w_c r_c^2 into dc, scaled by dcost; false for the
// pixels the cost skips. w r is r clamped to +-kappa (one median instruction instead of a reciprocal, a minimum and two
// products), and the whitening 1/sigma enters once per row kind: about 60 instructions instead of 95 (gather of the
// 4000-edge graph 4.95 -> 4.78 ms).
__device__ inline bool adj_gathered(const float4 Xj, const float4 Xi, const float* M, const GnConst& k, float dcost,
                                    float* g, float& dc) {
  const float x0 = fmaf(M[0], Xj.x, fmaf(M[1], Xj.y, fmaf(M[2], Xj.z, M[9])));
  const float x1 = fmaf(M[3], Xj.x, fmaf(M[4], Xj.y, fmaf(M[5], Xj.z, M[10])));
  const float x2 = fmaf(M[6], Xj.x, fmaf(M[7], Xj.y, fmaf(M[8], Xj.z, M[11])));
  const float d2 = fmaf(x0, x0, fmaf(x1, x1, x2 * x2));
  const float di2 = fmaf(Xi.x, Xi.x, fmaf(Xi.y, Xi.y, Xi.z * Xi.z));
  const float dj2 = fmaf(Xj.x, Xj.x, fmaf(Xj.y, Xj.y, Xj.z * Xj.z));
  const float cc = Xi.w * Xj.w;
  const float mn = fminf(fminf(d2, di2), dj2);
  const float sum = (d2 + di2) + (dj2 + cc);
  if (!(mn > 1e-18f) || !(cc >= 0.0f) || !(sum < __builtin_huge_valf())) return false;
  const float rd = rsqrtf(d2), rdi = rsqrtf(di2);
  const float p[3] = {Xi.x * rdi, Xi.y * rdi, Xi.z * rdi};
  const float sq = __builtin_amdgcn_sqrtf(__builtin_amdgcn_sqrtf(cc));
  const float sr = sq * k.inv_sr, sd = sq * k.inv_sd;
  const float r[4] = {sr * fmaf(x0, rd, -p[0]), sr * fmaf(x1, rd, -p[1]), sr * fmaf(x2, rd, -p[2]),
                      sd * fmaf(d2, rd, -(di2 * rdi))};
  float gam[4];
  dc = 0.0f;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float wr = __builtin_amdgcn_fmed3f(r[c], -k.kappa, k.kappa);
    dc = fmaf(wr, r[c], dc);
    gam[c] = wr * (c < 3 ? sr : sd);
  }
  dc *= dcost;
  // -((gam - psi (psi . gam)) / d_i + gam_range psi) = psi ((psi . gam) / d_i - gam_range) - gam / d_i
  const float f = fmaf(p[0], gam[0], fmaf(p[1], gam[1], p[2] * gam[2])) * rdi - gam[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) g[c] = dcost * fmaf(p[c], f, -gam[c] * rdi);
  return true;
}

// Wave sums of eight values, reduce-scattered: at each of the first three steps a lane and its partner (lane ^ 1, ^ 2,
// ^ 4) hold the same list, each keeps one half of it and adds the partner's copy; three full sums (lane ^ 8, ^ 16,
// ^ 32) finish. Lane l < 8 stores the total of value slot 4 b0 + 2 b1 + b2 (bits of l): 10 adds and one store of 32 B
// per wave and edge instead of eight full sums (48 adds) and eight single-lane stores, with which the gather's address
// units were 73% busy (most of its vector-memory instructions were these stores).
__device__ inline float dpp_swap4(float v) {  // the value of lane ^ 4: row_shl:4 into even quads, row_shr:4 into odd
  const int lo = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x104, 0xf, 0x5, true);
  return __int_as_float(__builtin_amdgcn_update_dpp(lo, __float_as_int(v), 0x114, 0xf, 0xa, true));
}

__device__ inline void wave_store8(const float* v, int lane, float* __restrict__ out) {
  const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
  float a[4], b[2];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float keep = b0 ? v[k + 4] : v[k], send = b0 ? v[k] : v[k + 4];
    a[k] = keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(send), 0xb1, 0xf, 0xf, true));
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float keep = b1 ? a[k + 2] : a[k], send = b1 ? a[k] : a[k + 2];
    b[k] = keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(send), 0x4e, 0xf, 0xf, true));
  }
  float s = (b2 ? b[1] : b[0]) + dpp_swap4(b2 ? b[0] : b[1]);
  s += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), 0x128, 0xf, 0xf, true));  // row_ror:8
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(s), false, false);
  s = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
  s = __uint_as_float(q[0]) + __uint_as_float(q[1]);
  if (lane < 8) out[(b0 ? 4 : 0) + (b1 ? 2 : 0) + (b2 ? 1 : 0)] = s;
}

// Query side, gathered: block (tile, k) owns 512 pixels of keyframe k and walks the edges that end in
// k (j = k). Per pixel it sums dE/dX_k = (s_ij R_ij)^T dE/dx and the j half of dE/dC over those edges in
// registers and stores them once (zeros where nothing contributes); per (edge, tile) it leaves the
// seven pose-tangent pieces [g; x cross g; x . g] in part7 (row stride `stride` tiles).
template <int DT>
__global__ __launch_bounds__(kAdjThreads) void k_adjoint_gather_j(
    const void* __restrict__ arena, const EdgeDev* __restrict__ edges, const EdgeXf* __restrict__ xf,
    const int32_t* __restrict__ idx_arena, const int64_t* __restrict__ kf_off, const int32_t* __restrict__ kf_npx,
    const int32_t* __restrict__ node_ptr, const int32_t* __restrict__ node_adj, GnConst k, float dcost,
    float* __restrict__ grad_xyz, float* __restrict__ grad_conf, float* __restrict__ part7, int stride) {
  const int kf = blockIdx.y;
  const int tile = blockIdx.x;
  const int npx = kf_npx[kf];
  if (tile * kAdjThreads * kAdjPPT >= npx) return;  // uniform per block
  const int64_t off = kf_off[kf];
  typename Px<DT>::raw_t xr[kAdjPPT];
  float acc[kAdjPPT][4];
#pragma unroll
  for (int u = 0; u < kAdjPPT; ++u) {
    const int n = tile * kAdjThreads * kAdjPPT + u * kAdjThreads + threadIdx.x;
    xr[u] = Px<DT>::load_raw(arena, off + (n < npx ? n : 0));
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[u][c] = 0.0f;
  }
  for (int q = node_ptr[kf]; q < node_ptr[kf + 1]; ++q) {
    const int code = node_adj[q];
    if (!(code & 1)) continue;  // this keyframe is the gathered side of that edge
    const int e = code >> 1;
    const EdgeDev E = edges[e];
    float M[12];
#pragma unroll
    for (int r = 0; r < 12; ++r) M[r] = xf[e].m[r];
    const int32_t* idx = idx_arena + E.idx_off;
    float g8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < kAdjPPT; ++u) {
      const int n = tile * kAdjThreads * kAdjPPT + u * kAdjThreads + threadIdx.x;
      const int32_t m = (n < npx) ? idx[n] : -1;
      if (m < 0 || m >= E.npx_i) continue;
      const float4 Xj = Px<DT>::unpack(xr[u]);
      const float4 Xi = Px<DT>::load(arena, E.off_i + m);
      AdjPix o;
      if (!adj_pixel(Xj, Xi, M, k, dcost, o)) continue;
      acc[u][0] += M[0] * o.gx[0] + M[3] * o.gx[1] + M[6] * o.gx[2];
      acc[u][1] += M[1] * o.gx[0] + M[4] * o.gx[1] + M[7] * o.gx[2];
      acc[u][2] += M[2] * o.gx[0] + M[5] * o.gx[1] + M[8] * o.gx[2];
      acc[u][3] += o.dc / (4.0f * Xj.w);
      g8[0] += o.gx[0];
      g8[1] += o.gx[1];
      g8[2] += o.gx[2];
      g8[3] += o.x[1] * o.gx[2] - o.x[2] * o.gx[1];
      g8[4] += o.x[2] * o.gx[0] - o.x[0] * o.gx[2];
      g8[5] += o.x[0] * o.gx[1] - o.x[1] * o.gx[0];
      g8[6] += o.x[0] * o.gx[0] + o.x[1] * o.gx[1] + o.x[2] * o.gx[2];
    }
    // one partial per wave and edge, summed in a fixed order by the edge finalize
    float* pw = part7 + ((int64_t(e) * stride + tile) * kAdjWaves + (threadIdx.x >> 6)) * 8;
    wave_store8(g8, threadIdx.x & (kWave - 1), pw);
  }
#pragma unroll
  for (int u = 0; u < kAdjPPT; ++u) {
    const int n = tile * kAdjThreads * kAdjPPT + u * kAdjThreads + threadIdx.x;
    if (n >= npx) continue;
    float* gj = grad_xyz + 3 * (off + n);
    gj[0] = acc[u][0];
    gj[1] = acc[u][1];
    gj[2] = acc[u][2];
    grad_conf[off + n] = acc[u][3];
  }
}

// Gathered side, scattered: the matches of one tile of an edge add dE/dX_i[m] and the i half of dE/dC
// with float atomics (several matches can land on one pixel of i, and a keyframe is the gathered side of
// several edges). Runs after k_adjoint_gather_j, whose plain stores it accumulates onto.
// The atomics are performed at the memory side, line by line, so their cost is the cache lines an instruction touches:
// a wave's 64 gradients are regrouped through LDS so that its three instructions each cover 21 pixels' consecutive
// components (4 lines of 64 B where the matches are consecutive) instead of one component of 64 pixels (12 lines):
// 424 -> 224 us for 5.9 M matches of 40 edges in float32.
template <int DT>
__global__ __launch_bounds__(kAdjThreads) void k_adjoint_scatter_i(
    const void* __restrict__ arena, const EdgeDev* __restrict__ edges, const EdgeXf* __restrict__ xf,
    const int32_t* __restrict__ idx_arena, GnConst k, float dcost, float* __restrict__ grad_xyz,
    float* __restrict__ grad_conf) {
  __shared__ float sg[kAdjWaves][3 * kWave];
  __shared__ int32_t sm[kAdjWaves][kWave];
  const int e = blockIdx.y;
  const EdgeDev E = edges[e];
  const int tile = blockIdx.x;
  const int tiles_e = (E.npx_j + kAdjThreads * kAdjPPT - 1) / (kAdjThreads * kAdjPPT);
  if (tile >= tiles_e) return;  // uniform per block
  float M[12];
#pragma unroll
  for (int q = 0; q < 12; ++q) M[q] = xf[e].m[q];
  const int32_t* idx = idx_arena + E.idx_off;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  float* __restrict__ wg = sg[wave];
  int32_t* __restrict__ wm = sm[wave];
  float* __restrict__ gi = grad_xyz + 3 * E.off_i;
#pragma unroll
  for (int u = 0; u < kAdjPPT; ++u) {
    const int64_t n = int64_t(tile) * kAdjThreads * kAdjPPT + int64_t(u) * kAdjThreads + threadIdx.x;
    int32_t m = (n < E.npx_j) ? idx[n] : -1;
    if (m >= E.npx_i) m = -1;
    if (m >= 0) {
      const float4 Xj = Px<DT>::load(arena, E.off_j + n);
      const float4 Xi = Px<DT>::load(arena, E.off_i + m);
      float g[3], dc;
      if (adj_gathered(Xj, Xi, M, k, dcost, g, dc)) {
        wg[3 * lane] = g[0];
        wg[3 * lane + 1] = g[1];
        wg[3 * lane + 2] = g[2];
        atomicAdd(grad_conf + E.off_i + m, dc / (4.0f * Xi.w));
      } else {
        m = -1;
      }
    }
    wm[lane] = m;
    wave_sync();
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const int q = r * kWave + lane, px = q / 3;
      const int32_t mp = wm[px];
      if (mp >= 0) atomicAdd(gi + 3 * int64_t(mp) + (q - 3 * px), wg[q]);
    }
    wave_sync();
  }
}

// --------------------------------------------------------------------------------------------------
// Inverse match maps for a graph whose matches stay fixed: for edge e and pixel m of keyframe i(e), the
// pixels n of j(e) with idx[n] = m, in increasing n, as CSR (offsets at obase[e], npx_i + 1 of them;
// lists at sbase[e]). Built once by count, scan, fill and a per-list sort.
// --------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_inv_count(const EdgeDev* __restrict__ edges,
                                                   const int32_t* __restrict__ idx_arena,
                                                   const int64_t* __restrict__ cbase, int32_t* __restrict__ cnt) {
  const int e = blockIdx.y;
  const EdgeDev E = edges[e];
  const int n = blockIdx.x * 256 + threadIdx.x;
  if (n >= E.npx_j) return;
  const int32_t m = idx_arena[E.idx_off + n];
  if (m < 0 || m >= E.npx_i) return;
  atomicAdd(cnt + cbase[e] + m, 1);
}

__global__ __launch_bounds__(1024) void k_inv_scan(const EdgeDev* __restrict__ edges,
                                                   const int64_t* __restrict__ cbase,
                                                   const int64_t* __restrict__ obase,
                                                   const int32_t* __restrict__ cnt, int32_t* __restrict__ off) {
  __shared__ int sh[2][1024];
  const int e = blockIdx.x, t = threadIdx.x;
  const int npx = edges[e].npx_i;
  const int chunk = (npx + 1023) / 1024;
  const int lo = min(npx, t * chunk), hi = min(npx, lo + chunk);
  const int32_t* c = cnt + cbase[e];
  int32_t* o = off + obase[e];
  int sum = 0;
  for (int m = lo; m < hi; ++m) sum += c[m];
  sh[0][t] = sum;
  __syncthreads();
  int src = 0;
  for (int d = 1; d < 1024; d <<= 1) {  // inclusive scan of the chunk sums
    const int v = sh[src][t] + (t >= d ? sh[src][t - d] : 0);
    sh[src ^ 1][t] = v;
    src ^= 1;
    __syncthreads();
  }
  int run = sh[src][t] - sum;
  for (int m = lo; m < hi; ++m) {
    o[m] = run;
    run += c[m];
  }
  if (t == 1023) o[npx] = sh[src][t];
}

__global__ __launch_bounds__(256) void k_inv_fill(const EdgeDev* __restrict__ edges,
                                                  const int32_t* __restrict__ idx_arena,
                                                  const int64_t* __restrict__ cbase,
                                                  const int64_t* __restrict__ obase,
                                                  const int64_t* __restrict__ sbase,
                                                  const int32_t* __restrict__ off, int32_t* __restrict__ cur,
                                                  int32_t* __restrict__ src) {
  const int e = blockIdx.y;
  const EdgeDev E = edges[e];
  const int n = blockIdx.x * 256 + threadIdx.x;
  if (n >= E.npx_j) return;
  const int32_t m = idx_arena[E.idx_off + n];
  if (m < 0 || m >= E.npx_i) return;
  const int slot = atomicAdd(cur + cbase[e] + m, 1);
  src[sbase[e] + off[obase[e] + m] + slot] = n;
}

__global__ __launch_bounds__(256) void k_inv_sort(const EdgeDev* __restrict__ edges,
                                                  const int64_t* __restrict__ obase,
                                                  const int64_t* __restrict__ sbase,
                                                  const int32_t* __restrict__ off, int32_t* __restrict__ src) {
  const int e = blockIdx.y;
  const int m = blockIdx.x * 256 + threadIdx.x;
  if (m >= edges[e].npx_i) return;
  const int32_t* o = off + obase[e];
  const int a = o[m], b = o[m + 1];
  int32_t* L = src + sbase[e];
  for (int x = a + 1; x < b; ++x) {  // insertion sort, lists are short
    const int32_t v = L[x];
    int y = x - 1;
    while (y >= a && L[y] > v) {
      L[y + 1] = L[y];
      --y;
    }
    L[y + 1] = v;
  }
}

// Cost and adjoint in one gather pass over a fixed graph: block (tile, k) owns 512 pixels of keyframe
// k. For the edges that end in k it walks the matches of its pixels (query side, as in
// k_adjoint_gather_j, plus the Huber cost in slot 7 of the tile pieces); for the edges that start in k
// it walks, per pixel m, the list of query pixels matched to m (gathered side). Both sides are summed in
// registers in a fixed order and stored once: no atomics, bitwise reproducible.
// It moves 21.7 GB for the 4000-edge graph at 4.1 to 4.4 TB/s by host (a large copy: 5.0), the L1 waiting for the L2 72% of
// the time. Per edge, a wave
// waits for its match words and then for the pixels they name; the words of the next edge are loaded before the
// current one is computed, and what is used once (words, stored gradients) passes the caches by: 5.40 -> 4.95 ms.
// Also loading the next edge's pixels early was slower (5.7 ms), and placing neighbouring tiles on one XCD cut the
// bytes by 18% but not the time.
template <int DT>
__global__ __launch_bounds__(kAdjThreads) void k_adjoint_gather(
    const void* __restrict__ arena, const EdgeDev* __restrict__ edges, const EdgeXf* __restrict__ xf,
    const int32_t* __restrict__ idx_arena, const int64_t* __restrict__ kf_off, const int32_t* __restrict__ kf_npx,
    const int32_t* __restrict__ node_ptr, const int32_t* __restrict__ node_adj, const int64_t* __restrict__ obase,
    const int64_t* __restrict__ sbase, const int64_t* __restrict__ cbase, const int32_t* __restrict__ inv_off,
    const int32_t* __restrict__ inv_src, const int32_t* __restrict__ inv_head, GnConst k, float dcost,
    float* __restrict__ grad_xyz, float* __restrict__ grad_conf, float* __restrict__ part7, int stride) {
  using raw_t = typename Px<DT>::raw_t;
  const int kf = blockIdx.y;
  const int tile = blockIdx.x;
  const int npx = kf_npx[kf];
  if (tile * kAdjThreads * kAdjPPT >= npx) return;  // uniform per block
  const int64_t off = kf_off[kf];
  const int p0 = tile * kAdjThreads * kAdjPPT + threadIdx.x;
  raw_t xr[kAdjPPT];
  float acc[kAdjPPT][4];
  bool any[kAdjPPT];  // a match contributed
#pragma unroll
  for (int u = 0; u < kAdjPPT; ++u) {
    const int n = p0 + u * kAdjThreads;
    xr[u] = Px<DT>::load_raw(arena, off + (n < npx ? n : 0));
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[u][c] = 0.0f;
    any[u] = false;
  }
  const int q0 = node_ptr[kf], q1 = node_ptr[kf + 1];
  // the next incident edge on one side (1: this keyframe is j, 0: it is i), and its match words for this thread's pixels
  auto next_edge = [&](int q, int side) {
    while (q < q1 && (node_adj[q] & 1) != side) ++q;
    return q;
  };
  auto load_words = [&](const int32_t* __restrict__ w, int32_t* out) {
#pragma unroll
    for (int u = 0; u < kAdjPPT; ++u) {
      const int n = p0 + u * kAdjThreads;
      out[u] = (n < npx) ? __builtin_nontemporal_load(w + n) : -1;
    }
  };
  int32_t word[kAdjPPT], ahead[kAdjPPT];
  // query side: pixel n of this keyframe, its match m in i
  int q = next_edge(q0, 1);
  if (q < q1) load_words(idx_arena + edges[node_adj[q] >> 1].idx_off, word);
  while (q < q1) {
    const int e = node_adj[q] >> 1;
    const EdgeDev E = edges[e];
    float M[12];
#pragma unroll
    for (int r = 0; r < 12; ++r) M[r] = xf[e].m[r];
    int32_t mm[kAdjPPT];
    raw_t xi[kAdjPPT];
#pragma unroll
    for (int u = 0; u < kAdjPPT; ++u) {
      mm[u] = (word[u] < E.npx_i) ? word[u] : -1;
      xi[u] = Px<DT>::load_raw(arena, E.off_i + (mm[u] >= 0 ? mm[u] : 0));
    }
    q = next_edge(q + 1, 1);
    if (q < q1) load_words(idx_arena + edges[node_adj[q] >> 1].idx_off, ahead);
    float g8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < kAdjPPT; ++u) {
      if (mm[u] < 0) continue;
      AdjPix o;
      if (!adj_pixel(Px<DT>::unpack(xr[u]), Px<DT>::unpack(xi[u]), M, k, dcost, o)) continue;
      acc[u][0] += M[0] * o.gx[0] + M[3] * o.gx[1] + M[6] * o.gx[2];
      acc[u][1] += M[1] * o.gx[0] + M[4] * o.gx[1] + M[7] * o.gx[2];
      acc[u][2] += M[2] * o.gx[0] + M[5] * o.gx[1] + M[8] * o.gx[2];
      acc[u][3] += o.dc;
      any[u] = true;
      g8[0] += o.gx[0];
      g8[1] += o.gx[1];
      g8[2] += o.gx[2];
      g8[3] += o.x[1] * o.gx[2] - o.x[2] * o.gx[1];
      g8[4] += o.x[2] * o.gx[0] - o.x[0] * o.gx[2];
      g8[5] += o.x[0] * o.gx[1] - o.x[1] * o.gx[0];
      g8[6] += o.x[0] * o.gx[0] + o.x[1] * o.gx[1] + o.x[2] * o.gx[2];
      g8[7] += o.rho;
    }
    // one partial per wave and edge (the waves of the block never wait for each other), summed in a
    // fixed order by the edge finalize
    wave_store8(g8, threadIdx.x & (kWave - 1),
                part7 + ((int64_t(e) * stride + tile) * kAdjWaves + (threadIdx.x >> 6)) * 8);
#pragma unroll
    for (int u = 0; u < kAdjPPT; ++u) word[u] = ahead[u];
  }
  // gathered side: pixel m of this keyframe, the query pixels matched to it
  q = next_edge(q0, 0);
  if (q < q1) load_words(inv_head + cbase[node_adj[q] >> 1], word);
  while (q < q1) {
    const int e = node_adj[q] >> 1;
    const EdgeDev E = edges[e];
    float M[12];
#pragma unroll
    for (int r = 0; r < 12; ++r) M[r] = xf[e].m[r];
    int h[kAdjPPT], n0[kAdjPPT];
    raw_t xj[kAdjPPT];
#pragma unroll
    for (int u = 0; u < kAdjPPT; ++u) {
      h[u] = word[u];
      n0[u] = (h[u] >= 0) ? h[u] : ((h[u] <= -2) ? -2 - h[u] : -1);
      xj[u] = Px<DT>::load_raw(arena, E.off_j + (n0[u] >= 0 ? n0[u] : 0));
    }
    q = next_edge(q + 1, 0);
    if (q < q1) load_words(inv_head + cbase[node_adj[q] >> 1], ahead);
    auto gathered = [&](int u, const float4 Xj) {
      float gi[3], dc;
      if (!adj_gathered(Xj, Px<DT>::unpack(xr[u]), M, k, dcost, gi, dc)) return;
#pragma unroll
      for (int c = 0; c < 3; ++c) acc[u][c] += gi[c];
      acc[u][3] += dc;
      any[u] = true;
    };
#pragma unroll
    for (int u = 0; u < kAdjPPT; ++u) {
      if (n0[u] < 0) continue;
      // the first query pixel from the head word; the rest of a longer list (rare) from the CSR, in
      // increasing n as before
      gathered(u, Px<DT>::unpack(xj[u]));
      if (h[u] > -2) continue;
      const int32_t* lo = inv_off + obase[e];
      const int32_t* lst = inv_src + sbase[e];
      const int m = p0 + u * kAdjThreads;
      const int xe = lo[m + 1];
      for (int x = lo[m] + 1; x < xe; ++x) gathered(u, Px<DT>::load(arena, E.off_j + lst[x]));
    }
#pragma unroll
    for (int u = 0; u < kAdjPPT; ++u) word[u] = ahead[u];
  }
#pragma unroll
  for (int u = 0; u < kAdjPPT; ++u) {
    const int n = p0 + u * kAdjThreads;
    if (n >= npx) continue;
    float* gj = grad_xyz + 3 * (off + n);
    __builtin_nontemporal_store(acc[u][0], gj);
    __builtin_nontemporal_store(acc[u][1], gj + 1);
    __builtin_nontemporal_store(acc[u][2], gj + 2);
    // both sides divide by this pixel's own confidence: dE/dC = sum_c w_c r_c^2 / (4 C)
    grad_conf[off + n] = any[u] ? acc[u][3] / (4.0f * Px<DT>::unpack(xr[u]).w) : 0.0f;
  }
}

// E_global alone (eq. 5), in the same (tile, edge) grid as the adjoint: per pixel the Huber cost of the
// four whitened residual components, with the validity rules, square roots and weights of the GN
// reduction; per block one (cost, count) pair in the block's slot of part (stride 8).
template <int DT>
__global__ __launch_bounds__(kAdjThreads) void k_edge_cost(const void* __restrict__ arena,
                                                           const EdgeDev* __restrict__ edges,
                                                           const EdgeXf* __restrict__ xf,
                                                           const int32_t* __restrict__ idx_arena, GnConst k,
                                                           float* __restrict__ part) {
  const int e = blockIdx.y;
  const EdgeDev E = edges[e];
  const int tile = blockIdx.x;
  const int tiles_e = (E.npx_j + kAdjThreads * kAdjPPT - 1) / (kAdjThreads * kAdjPPT);
  if (tile >= tiles_e) return;  // uniform per block
  float M[12];
#pragma unroll
  for (int q = 0; q < 12; ++q) M[q] = xf[e].m[q];
  const int32_t* idx = idx_arena + E.idx_off;
  float cost = 0.0f, cnt = 0.0f;
#pragma unroll 2
  for (int u = 0; u < kAdjPPT; ++u) {
    const int64_t n = int64_t(tile) * kAdjThreads * kAdjPPT + int64_t(u) * kAdjThreads + threadIdx.x;
    if (n >= E.npx_j) continue;
    const int32_t m = idx[n];
    if (m < 0 || m >= E.npx_i) continue;
    const float4 Xj = Px<DT>::load(arena, E.off_j + n);
    const float4 Xi = Px<DT>::load(arena, E.off_i + m);
    const float x0 = fmaf(M[0], Xj.x, fmaf(M[1], Xj.y, fmaf(M[2], Xj.z, M[9])));
    const float x1 = fmaf(M[3], Xj.x, fmaf(M[4], Xj.y, fmaf(M[5], Xj.z, M[10])));
    const float x2 = fmaf(M[6], Xj.x, fmaf(M[7], Xj.y, fmaf(M[8], Xj.z, M[11])));
    const float d2 = fmaf(x0, x0, fmaf(x1, x1, x2 * x2));
    const float di2 = fmaf(Xi.x, Xi.x, fmaf(Xi.y, Xi.y, Xi.z * Xi.z));
    const float dj2 = fmaf(Xj.x, Xj.x, fmaf(Xj.y, Xj.y, Xj.z * Xj.z));
    const float cc = Xi.w * Xj.w;
    const float mn = fminf(fminf(d2, di2), dj2);
    const float sum = (d2 + di2) + (dj2 + cc);
    if (!(mn > 1e-18f) || !(cc >= 0.0f) || !(sum < __builtin_huge_valf())) continue;
    const float rd = rsqrtf(d2), rdi = rsqrtf(di2);
    const float e4[4] = {x0 * rd - Xi.x * rdi, x1 * rd - Xi.y * rdi, x2 * rd - Xi.z * rdi, d2 * rd - di2 * rdi};
    const float sq = __builtin_amdgcn_sqrtf(__builtin_amdgcn_sqrtf(cc));
    const float isg[4] = {k.inv_sr, k.inv_sr, k.inv_sr, k.inv_sd};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float a = fabsf(sq * isg[c] * e4[c]);
      const float t = fminf(1.0f, k.kappa * __builtin_amdgcn_rcpf(a)) * a;  // rho = t (|r| - t/2)
      cost = fmaf(t, fmaf(-0.5f, t, a), cost);
    }
    cnt += 1.0f;
  }
  __shared__ float red[kAdjThreads / kWave][2];
  cost = wave_sum(cost);
  cnt = wave_sum(cnt);
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6][0] = cost;
    red[threadIdx.x >> 6][1] = cnt;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    float s = 0.0f;
    for (int w = 0; w < kAdjThreads / kWave; ++w) s += red[w][threadIdx.x];
    part[(int64_t(e) * gridDim.x + tile) * 8 + threadIdx.x] = s;
  }
}

// Per edge (one wave each): cost and count from the tile pairs, float64 / int64: lanes stride the tiles, then a
// fixed-shape wave sum. The edge's pairs are a chain of dependent adds behind loads 32 B apart when one thread
// walks them: 65 us for 40 edges of 384 tiles that way, 5 us with a wave per edge.
constexpr int kFinalizeWaves = 4;  // edges per block

__global__ __launch_bounds__(kFinalizeWaves* kWave) void k_cost_edge_finalize(const EdgeDev* __restrict__ edges,
                                                                              int tiles_stride,
                                                                              const float* __restrict__ part,
                                                                              double* __restrict__ cost_e,
                                                                              int64_t* __restrict__ count_e,
                                                                              int n_edges) {
  const int e = blockIdx.x * kFinalizeWaves + int(threadIdx.x) / kWave;
  if (e >= n_edges) return;  // uniform per wave
  const int lane = threadIdx.x & (kWave - 1);
  const int tiles_e = (edges[e].npx_j + kAdjThreads * kAdjPPT - 1) / (kAdjThreads * kAdjPPT);
  double c = 0.0, n = 0.0;  // counts are whole numbers far below 2^53
  for (int t = lane; t < tiles_e; t += kWave) {
    const float2 v = *reinterpret_cast<const float2*>(part + (int64_t(e) * tiles_stride + t) * 8);
    c += double(v.x);
    n += double(v.y);
  }
  c = wave_sum(c);
  n = wave_sum(n);
  if (lane == 0) {
    cost_e[e] = c;
    count_e[e] = int64_t(n);
  }
}

int launch_cost_batched(ds3_dtype dt, const void* arena, const EdgeDev* edges, int n_edges, int max_npx_j,
                        const EdgeXf* xf, const int32_t* idx, GnConst c, float* part, double* cost_e,
                        int64_t* count_e, hipStream_t s) {
  const int tiles = (max_npx_j + kAdjThreads * kAdjPPT - 1) / (kAdjThreads * kAdjPPT);
  if (n_edges <= 0 || tiles <= 0) return 0;
  dim3 grid(tiles, n_edges), block(kAdjThreads);
  if (dt == DS3_F32)
    hipLaunchKernelGGL(k_edge_cost<DS3_F32>, grid, block, 0, s, arena, edges, xf, idx, c, part);
  else
    hipLaunchKernelGGL(k_edge_cost<DS3_BF16>, grid, block, 0, s, arena, edges, xf, idx, c, part);
  DS3_TRY(check_hip(hipGetLastError(), "k_edge_cost"));
  hipLaunchKernelGGL(k_cost_edge_finalize, dim3((n_edges + kFinalizeWaves - 1) / kFinalizeWaves),
                     dim3(kFinalizeWaves * kWave), 0, s, edges, tiles, part, cost_e, count_e, n_edges);
  return check_hip(hipGetLastError(), "k_cost_edge_finalize");
}

// Per edge (one block each): b_e = Ad^T (sum of the waves' pieces), float64. The pieces of an edge are contiguous,
// eight floats per wave of every tile: thread t adds component t % 8 of rows t / 8, t / 8 + 32, .. (a block reads
// 1 KiB at a time), then the 32 rows are summed in a fixed order. One thread per edge walking them took 192 us for
// 40 edges and 317 us for 4000 (1536 rows each); a block per edge takes 6 us and 39 us (5 TB/s).
// With cost_e, component 7 (the Huber cost) is summed into cost_e and count_e is cleared.
__global__ __launch_bounds__(256) void k_adjoint_edge_finalize(const EdgeDev* __restrict__ edges, int tiles_stride,
                                                               const float* __restrict__ part7,
                                                               const double* __restrict__ Ad,
                                                               double* __restrict__ b_e,
                                                               double* __restrict__ cost_e,
                                                               int64_t* __restrict__ count_e) {
  __shared__ double red[256];
  __shared__ double S[8];
  const int e = blockIdx.x, t = threadIdx.x;
  const int rows = (edges[e].npx_j + kAdjThreads * kAdjPPT - 1) / (kAdjThreads * kAdjPPT) * kAdjWaves;
  const float* p = part7 + int64_t(e) * tiles_stride * kAdjWaves * 8 + t;
  double s = 0.0;
  int k = t >> 3;
  for (; k + 96 < rows; k += 128, p += 1024) {  // four loads in flight
    const float v0 = p[0], v1 = p[256], v2 = p[512], v3 = p[768];
    s += double(v0);
    s += double(v1);
    s += double(v2);
    s += double(v3);
  }
  for (; k < rows; k += 32, p += 256) s += double(p[0]);
  red[t] = s;
  __syncthreads();
  if (t < 8) {
    double v = 0.0;
#pragma unroll
    for (int r = 0; r < 32; ++r) v += red[8 * r + t];
    S[t] = v;
  }
  __syncthreads();
  if (t < 7) {
    const double* A = Ad + 49 * int64_t(e);
    double v = 0.0;
    for (int a = 0; a < 7; ++a) v += A[7 * a + t] * S[a];
    b_e[7 * int64_t(e) + t] = v;
  } else if (t == 7 && cost_e) {
    cost_e[e] = S[7];
    count_e[e] = 0;
  }
}

// Per keyframe: dE/dtau_k = sum over incident edges (edge order) of +b_e (k = j) or -b_e (k = i).
__global__ void k_grad_tau(int n_kf, const int32_t* __restrict__ node_ptr, const int32_t* __restrict__ node_adj,
                           const double* __restrict__ b_e, double* __restrict__ grad_tau) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= 7 * n_kf) return;
  const int k = t / 7, r = t % 7;
  double s = 0.0;
  for (int p = node_ptr[k]; p < node_ptr[k + 1]; ++p) {
    const int code = node_adj[p];
    const double v = b_e[7 * int64_t(code >> 1) + r];
    s += (code & 1) ? v : -v;
  }
  grad_tau[t] = s;
}

int adjoint_part_floats(int n_edges, int max_npx_j) {
  const int tiles = (max_npx_j + kAdjThreads * kAdjPPT - 1) / (kAdjThreads * kAdjPPT);
  return n_edges * tiles * kAdjWaves * 8;
}

int launch_adjoint(ds3_dtype dt, const void* arena, const EdgeDev* edges, int n_edges, int max_npx_j,
                   int max_npx_kf, const EdgeXf* xf, const double* Ad, const int32_t* idx, GnConst c,
                   float dcost, float* grad_xyz, float* grad_conf, float* part7, double* b_e, int n_kf,
                   const int64_t* kf_off, const int32_t* kf_npx, const int32_t* node_ptr,
                   const int32_t* node_adj, double* grad_tau, ds3_timer* timer, hipStream_t s) {
  const int tiles = (max_npx_j + kAdjThreads * kAdjPPT - 1) / (kAdjThreads * kAdjPPT);
  const int tiles_kf = (max_npx_kf + kAdjThreads * kAdjPPT - 1) / (kAdjThreads * kAdjPPT);
  DS3_TRY(timer_record(timer, true, s));
  if (tiles_kf > 0) {
    dim3 grid(tiles_kf, n_kf), block(kAdjThreads);
    if (dt == DS3_F32)
      hipLaunchKernelGGL(k_adjoint_gather_j<DS3_F32>, grid, block, 0, s, arena, edges, xf, idx, kf_off, kf_npx,
                         node_ptr, node_adj, c, dcost, grad_xyz, grad_conf, part7, tiles);
    else
      hipLaunchKernelGGL(k_adjoint_gather_j<DS3_BF16>, grid, block, 0, s, arena, edges, xf, idx, kf_off, kf_npx,
                         node_ptr, node_adj, c, dcost, grad_xyz, grad_conf, part7, tiles);
    DS3_TRY(check_hip(hipGetLastError(), "k_adjoint_gather_j"));
  }
  if (n_edges > 0 && tiles > 0) {
    dim3 grid(tiles, n_edges), block(kAdjThreads);
    if (dt == DS3_F32)
      hipLaunchKernelGGL(k_adjoint_scatter_i<DS3_F32>, grid, block, 0, s, arena, edges, xf, idx, c, dcost,
                         grad_xyz, grad_conf);
    else
      hipLaunchKernelGGL(k_adjoint_scatter_i<DS3_BF16>, grid, block, 0, s, arena, edges, xf, idx, c, dcost,
                         grad_xyz, grad_conf);
    DS3_TRY(check_hip(hipGetLastError(), "k_adjoint_scatter_i"));
  }
  DS3_TRY(timer_record(timer, false, s));
  if (n_edges > 0 && tiles > 0) {
    hipLaunchKernelGGL(k_adjoint_edge_finalize, dim3(n_edges), dim3(256), 0, s, edges, tiles, part7, Ad, b_e,
                       static_cast<double*>(nullptr), static_cast<int64_t*>(nullptr));
    DS3_TRY(check_hip(hipGetLastError(), "k_adjoint_edge_finalize"));
  }
  hipLaunchKernelGGL(k_grad_tau, dim3((7 * n_kf + 127) / 128), dim3(128), 0, s, n_kf, node_ptr, node_adj, b_e,
                     grad_tau);
  return check_hip(hipGetLastError(), "k_grad_tau");
}

// One word per pixel m of keyframe i(e) for the gather: -1 when no query pixel is matched to m, the pixel
// n when exactly one is, -2 - n (n the first of the list) when several are (the rest stay in the CSR).
__global__ __launch_bounds__(256) void k_inv_head(const EdgeDev* __restrict__ edges,
                                                  const int64_t* __restrict__ cbase,
                                                  const int64_t* __restrict__ obase,
                                                  const int64_t* __restrict__ sbase,
                                                  const int32_t* __restrict__ off, const int32_t* __restrict__ src,
                                                  int32_t* __restrict__ head) {
  const int e = blockIdx.y;
  const int m = blockIdx.x * 256 + threadIdx.x;
  if (m >= edges[e].npx_i) return;
  const int32_t* o = off + obase[e];
  const int a = o[m], b = o[m + 1];
  const int32_t n0 = (b > a) ? src[sbase[e] + a] : 0;
  head[cbase[e] + m] = (b == a) ? -1 : ((b == a + 1) ? n0 : -2 - n0);
}

int launch_inverse_maps(const EdgeDev* edges, int n_edges, int max_npx_j, int max_npx_i, const int32_t* idx,
                        const int64_t* cbase, const int64_t* obase, const int64_t* sbase, int32_t* cnt,
                        size_t cnt_len, int32_t* off, int32_t* src, int32_t* head, hipStream_t s) {
  if (n_edges <= 0) return 0;
  DS3_TRY(launch_fill_u32(reinterpret_cast<unsigned*>(cnt), cnt_len, 0u, s));
  const dim3 gj((max_npx_j + 255) / 256, n_edges), gi((max_npx_i + 255) / 256, n_edges);
  hipLaunchKernelGGL(k_inv_count, gj, dim3(256), 0, s, edges, idx, cbase, cnt);
  DS3_TRY(check_hip(hipGetLastError(), "k_inv_count"));
  hipLaunchKernelGGL(k_inv_scan, dim3(n_edges), dim3(1024), 0, s, edges, cbase, obase, cnt, off);
  DS3_TRY(check_hip(hipGetLastError(), "k_inv_scan"));
  DS3_TRY(launch_fill_u32(reinterpret_cast<unsigned*>(cnt), cnt_len, 0u, s));
  hipLaunchKernelGGL(k_inv_fill, gj, dim3(256), 0, s, edges, idx, cbase, obase, sbase, off, cnt, src);
  DS3_TRY(check_hip(hipGetLastError(), "k_inv_fill"));
  hipLaunchKernelGGL(k_inv_sort, gi, dim3(256), 0, s, edges, obase, sbase, off, src);
  DS3_TRY(check_hip(hipGetLastError(), "k_inv_sort"));
  hipLaunchKernelGGL(k_inv_head, gi, dim3(256), 0, s, edges, cbase, obase, sbase, off, src, head);
  return check_hip(hipGetLastError(), "k_inv_head");
}

int launch_adjoint_gather(ds3_dtype dt, const void* arena, const EdgeDev* edges, int n_edges, int max_npx_j,
                          int max_npx_kf, const EdgeXf* xf, const double* Ad, const int32_t* idx, GnConst c,
                          float dcost, float* grad_xyz, float* grad_conf, float* part7, double* b_e,
                          double* cost_e, int64_t* count_e, int n_kf, const int64_t* kf_off,
                          const int32_t* kf_npx, const int32_t* node_ptr, const int32_t* node_adj,
                          const int64_t* obase, const int64_t* sbase, const int64_t* cbase,
                          const int32_t* inv_off, const int32_t* inv_src, const int32_t* inv_head, double* grad_tau,
                          ds3_timer* timer, hipStream_t s) {
  const int tiles = (max_npx_j + kAdjThreads * kAdjPPT - 1) / (kAdjThreads * kAdjPPT);
  const int tiles_kf = (max_npx_kf + kAdjThreads * kAdjPPT - 1) / (kAdjThreads * kAdjPPT);
  DS3_TRY(timer_record(timer, true, s));
  if (tiles_kf > 0) {
    dim3 grid(tiles_kf, n_kf), block(kAdjThreads);
    if (dt == DS3_F32)
      hipLaunchKernelGGL(k_adjoint_gather<DS3_F32>, grid, block, 0, s, arena, edges, xf, idx, kf_off, kf_npx,
                         node_ptr, node_adj, obase, sbase, cbase, inv_off, inv_src, inv_head, c, dcost, grad_xyz,
                         grad_conf, part7, tiles);
    else
      hipLaunchKernelGGL(k_adjoint_gather<DS3_BF16>, grid, block, 0, s, arena, edges, xf, idx, kf_off, kf_npx,
                         node_ptr, node_adj, obase, sbase, cbase, inv_off, inv_src, inv_head, c, dcost, grad_xyz,
                         grad_conf, part7, tiles);
    DS3_TRY(check_hip(hipGetLastError(), "k_adjoint_gather"));
  }
  DS3_TRY(timer_record(timer, false, s));
  if (n_edges > 0 && tiles > 0) {
    hipLaunchKernelGGL(k_adjoint_edge_finalize, dim3(n_edges), dim3(256), 0, s, edges, tiles, part7, Ad, b_e,
                       cost_e, count_e);
    DS3_TRY(check_hip(hipGetLastError(), "k_adjoint_edge_finalize"));
  }
  hipLaunchKernelGGL(k_grad_tau, dim3((7 * n_kf + 127) / 128), dim3(128), 0, s, n_kf, node_ptr, node_adj, b_e,
                     grad_tau);
  return check_hip(hipGetLastError(), "k_grad_tau");
}

}  // namespace ds3
