// The gradient step of a small dense network in one workgroup: Phases I, II and III one product after the other, with
// activations, cotangents and signs in LDS.
//
// A network of four layers of 64 on a batch of 32 is 17 launches of 2 to 6 us, each of them a launch, a memory latency and
// a few hundred clocks of work: 54 to 68 us, 56 here. A product is LDS reads, matrix instructions, epilogue and a
// barrier; its weights are loaded while the product before it runs. What bounds it is that chain on one CU: 2.9 us
// a layer in Phase I (1.0 without loads and matrix instructions, 0.7 for these, 1.0 for the loads, sixteen rows each of them), 2.1
// in Phase II, 8 in Phase III with two products and a weight gradient. The same products in the same order of k
// (gemm_fine.h), hence the bits of the launches layer by layer.
#include "gemm_fine.h"
#include "mw_internal.h"

namespace mw {

namespace {

constexpr int NT = 512, WAVES = NT / 64;
constexpr int KS = SMALL_NET_MAX_WIDTH / 32;   // slices of 32 k

// place of column n in a row of an LDS buffer: inside a slice of 32 in the order in which a lane reads its eight k
// (gemm_fine.h: lane group q has k = 16 (q & 1) + (q >> 1) + 0, 2, .. 14)
__device__ __forceinline__ int place(int n) { return (n & ~31) + (((n >> 4) & 1) + 2 * (n & 1)) * 8 + ((n & 15) >> 1); }

// The weights of one product for a wavefront's sixteen columns of the result, as they come from memory: nothing here waits for
// a load, so that they are on their way while the product before is formed (with the selection of a lane's k right
// behind its loads a layer took 4 us in Phase I).
struct Weights {
  float v[KS][16];

  // NT: element (k, n) at p[n K + k]. A lane takes sixteen k in a row and uses every other one of them (pick).
  __device__ __forceinline__ void load_nt(const float* __restrict__ p, int K, int N, int n, int q) {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(p, (uint32_t)(N * K) * 4u);
    const int k0 = 16 * (q & 1);
    if (K % 4 == 0) {
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = 32 * s + k0 + 4 * u;
          const float4 c = buf_load_f32x4(rs, n < N && k < K ? (uint32_t)(n * K + k) * 4u : OOB);
          v[s][4 * u] = c.x;
          v[s][4 * u + 1] = c.y;
          v[s][4 * u + 2] = c.z;
          v[s][4 * u + 3] = c.w;
        }
    } else {
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int k = 32 * s + k0 + (q >> 1) + 2 * i;
          v[s][2 * i] = buf_load_f32(rs, n < N && k < K ? (uint32_t)(n * K + k) * 4u : OOB);
          v[s][2 * i + 1] = v[s][2 * i];
        }
    }
  }
  // NN: element (k, n) at p[k N + n]
  __device__ __forceinline__ void load_nn(const float* __restrict__ p, int K, int N, int n, int q) {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(p, (uint32_t)(N * K) * 4u);
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = 32 * s + 16 * (q & 1) + (q >> 1) + 2 * i;
        v[s][2 * i] = buf_load_f32(rs, n < N && k < K ? (uint32_t)(k * N + n) * 4u : OOB);
        v[s][2 * i + 1] = v[s][2 * i];
      }
  }
  __device__ __forceinline__ float pick(int s, int i, int q) const { return (q >> 1) ? v[s][2 * i + 1] : v[s][2 * i]; }
};

// sixteen rows of an LDS buffer times the weights
__device__ __forceinline__ f32x4 product(const float* __restrict__ rows, int pitch, int K, const Weights& w, int r, int q) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    if (32 * s >= K) break;
    const float4* p = reinterpret_cast<const float4*>(rows + r * pitch + 32 * s + 8 * q);
    const float4 a = p[0], b = p[1];
    float fa[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    if (32 * s + 32 > K) {   // columns past the matrix may hold what an earlier, wider layer left there
#pragma unroll
      for (int i = 0; i < 8; ++i) fa[i] = 32 * s + 16 * (q & 1) + (q >> 1) + 2 * i < K ? fa[i] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i], w.pick(s, i, q), acc, 0, 0, 0);
  }
  return acc;
}

__global__ void __launch_bounds__(NT) k_small_net(SmallNet p) {
  extern __shared__ __align__(16) float lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int r = lane & 15, q = lane >> 4;
  const int B = p.B, L = p.L, pitch = p.pitch, size = p.rows * pitch, mtiles = (B + 15) / 16;
  float* const X = lds;                 // three buffers of activations (x_0 stays in the first until Phase III has used it)
  float* const H = lds + 3 * size;      // two of Phase III's cotangents
  float* const C = lds + 5 * size;      // two of pre-activation cotangents
  uint32_t* const bits = reinterpret_cast<uint32_t*>(lds + 7 * size);   // packed signs, layer after layer
  __shared__ double red[WAVES];

  // Columns a wavefront owns in a product: sixteen, in the row tiles m_first, m_first + m_step, ...
  int n_of = 0, m_first = 0, m_step = 1;
  auto split = [&](const SmallTiles& t) {
    n_of = (int)(t.at >> (4 * wave) & 15u) * 16 + r;
    m_first = (int)(t.round >> (4 * wave) & 15u);
    if (m_first >= t.groups) m_first = mtiles;   // (a wavefront too many has nothing to do)
    m_step = t.groups;
  };
  // the 32 packed signs around element (row, n) of layer l's output (any, outside), and which one it is
  auto sign_at = [&](const SmallLayer& l, int row, int n) {
    return row < B && n < l.d_out ? (uint32_t)row * (uint32_t)l.d_out + (uint32_t)n : 0u;
  };
  auto signs = [&](const SmallLayer& l, uint32_t e) { return bits[l.bits + (e >> 5)] >> (e & 31u); };

  Weights w, next;
  split(p.layer[0].out);
  w.load_nt(p.layer[0].W, p.layer[0].d_in, p.layer[0].d_out, n_of, q);
  // every line of the weights once, so that later loads find them in the nearest cache
  float touched = 0.f;
  for (int i = 0; i < L; ++i) {
    const SmallLayer& l = p.layer[i];
    const int n = l.d_in * l.d_out;
    for (int j = 32 * threadIdx.x; j < n; j += 32 * NT) touched += l.W[j] + l.P[j];
  }
  // all of LDS to zero: what lies outside a matrix must add nothing to a sum
  for (int i = 4 * threadIdx.x; i < 7 * size + p.bit_words; i += 4 * NT) *reinterpret_cast<float4*>(lds + i) = make_float4(0.f, 0.f, 0.f, 0.f);
  if (threadIdx.x < 3) p.status[threadIdx.x] = 0;
  __syncthreads();
  {
    const int d = p.layer[0].d_in;
    for (int row = wave; row < B; row += WAVES)
      for (int n = lane; n < d; n += 64) X[row * pitch + place(n)] = p.x[(int64_t)row * d + n];
  }
  __syncthreads();
  asm volatile("" ::"v"(touched));

  // ---- Phase I
  int xi = 0;
  for (int i = 0; i < L; ++i) {
    const SmallLayer& l = p.layer[i];
    split(l.out);
    const int n = n_of, m0 = m_first, step = m_step;
    if (i + 1 < L) {
      split(p.layer[i + 1].out);
      next.load_nt(p.layer[i + 1].W, p.layer[i + 1].d_in, p.layer[i + 1].d_out, n_of, q);
    } else {
      split(l.in);
      next.load_nn(l.W, l.d_out, l.d_in, n_of, q);
    }
    const int xo = i == 0 ? 1 : 3 - xi;   // 1, 2, 1, 2, ..
    const float bias = l.b && n < l.d_out ? l.b[n] : 0.f;
    for (int m = m0; m < mtiles; m += step) {
      const f32x4 acc = product(X + xi * size + m * 16 * pitch, pitch, l.d_in, w, r, q);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = m * 16 + 4 * q + j;
        const bool valid = row < B && n < l.d_out;
        float z = acc[j];
        if (l.b) z += bias;
        const bool bit = valid && z > 0.f;
        X[xo * size + row * pitch + place(n)] = valid ? (bit ? z : l.alpha * z) : 0.f;   // (rows up to a multiple of 32)
        // sixteen lanes hold a row's signs: the first two put them into the one or two words they lie in
        const uint32_t sixteen = (uint32_t)(__ballot(bit) >> (16 * q)) & 0xFFFFu;
        const uint32_t e = (uint32_t)row * (uint32_t)l.d_out + (uint32_t)(n - r), sh = e & 31u;
        const uint32_t part = r == 0 ? sixteen << sh : (sh > 16 ? sixteen >> (32 - sh) : 0u);
        if (r < 2 && part) atomicOr(&bits[l.bits + (e >> 5) + r], part);
      }
    }
    w = next;
    xi = xo;
    __syncthreads();
  }

  // ---- loss, the cotangent of the output and of its pre-activations
  {
    const SmallLayer& l = p.layer[L - 1];
    double sum = 0.0;
    for (int row = wave; row < B; row += WAVES)
      for (int n = lane; n < l.d_out; n += 64) {
        const float d = X[xi * size + row * pitch + place(n)] - p.target[(int64_t)row * l.d_out + n];
        sum += (double)d * (double)d;
        const float h = d * p.cot_scale;
        C[row * pitch + place(n)] = h * ((signs(l, sign_at(l, row, n)) & 1u) ? 1.f : l.alpha);
      }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if (lane == 0) red[wave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int i = 0; i < WAVES; ++i) t += red[i];
      const float v = (float)(p.loss_factor * t);
      if (p.loss) *p.loss = v;
      p.status[3] = fabsf(v) <= 3.402823466e38f ? 0u : 1u;   // NaN or infinity
    }
    for (int i = 0; i < L; ++i) {   // the signs, for whoever asks for them
      const SmallLayer& k = p.layer[i];
      const int words = (int)(((int64_t)B * k.d_out + 63) / 64) * 2;
      for (int j = threadIdx.x; j < words; j += NT) reinterpret_cast<uint32_t*>(k.mask)[j] = bits[k.bits + j];
    }
  }

  // ---- Phase II
  int ci = 0;
  for (int i = L - 1; i >= 0; --i) {
    const SmallLayer& l = p.layer[i];
    const int N = l.d_in;
    split(l.in);
    const int n = n_of, m0 = m_first, step = m_step;
    if (i > 0) {
      split(p.layer[i - 1].in);
      next.load_nn(p.layer[i - 1].W, p.layer[i - 1].d_out, p.layer[i - 1].d_in, n_of, q);
    } else {
      split(l.out);
      next.load_nt(l.W, l.d_in, l.d_out, n_of, q);
    }
    const SmallLayer& below = p.layer[i > 0 ? i - 1 : 0];
    for (int m = m0; m < mtiles; m += step) {
      const int row0 = m * 16 + 4 * q;
      uint32_t e[4], sg[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        e[j] = i > 0 ? sign_at(below, row0 + j, n) : 0u;
        sg[j] = signs(below, e[j]);
      }
      const f32x4 acc = product(C + ci * size + m * 16 * pitch, pitch, l.d_out, w, r, q);
      float* const raw = i == 0 ? p.h0 : below.ckpt;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool valid = row0 + j < B && n < N;
        const float h = acc[j];
        if (raw && valid) raw[(int64_t)(row0 + j) * N + n] = h;
        const int at = (row0 + j) * pitch + place(n);
        if (i == 0) H[at] = valid ? h : 0.f;
        else C[(1 - ci) * size + at] = valid ? h * ((sg[j] & 1u) ? 1.f : below.alpha) : 0.f;
      }
    }
    w = next;
    ci = 1 - ci;
    __syncthreads();
  }
  __syncthreads();   // checkpoints are read back below

  // ---- Phase III. A layer's weight gradient goes with the next layer's products: it reads buffers that those leave alone.
  Weights pw, next_pw;
  split(p.layer[0].out);
  pw.load_nt(p.layer[0].P, p.layer[0].d_in, p.layer[0].d_out, n_of, q);
  uint32_t mism = 0;
  xi = 0;
  int hi = 0;
  ci = 0;
  for (int i = 0; i <= L; ++i) {
    if (i < L) {
      const SmallLayer& l = p.layer[i];
      split(l.out);
      const int n = n_of, m0 = m_first, step = m_step;
      if (i + 1 < L) {
        const SmallLayer& up = p.layer[i + 1];
        split(up.out);
        next.load_nt(up.W, up.d_in, up.d_out, n_of, q);
        next_pw.load_nt(up.P, up.d_in, up.d_out, n_of, q);
      }
      const int xo = xi == 2 ? 0 : xi + 1;
      const float bias = l.b && n < l.d_out ? l.b[n] : 0.f, inv_alpha = 1.0f / l.alpha;
      for (int m = m0; m < mtiles; m += step) {
        uint32_t sg[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) sg[j] = signs(l, sign_at(l, m * 16 + 4 * q + j, n));
        const f32x4 az = product(X + xi * size + m * 16 * pitch, pitch, l.d_in, w, r, q);
        const f32x4 ac = product(H + hi * size + m * 16 * pitch, pitch, l.d_in, pw, r, q);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int row = m * 16 + 4 * q + j;
          const bool valid = row < B && n < l.d_out;
          float z = az[j];
          if (l.b) z += bias;
          const bool fresh = z > 0.f;
          if (valid && fresh != (bool)(sg[j] & 1u)) ++mism;
          const float c = ac[j];
          float h = fresh ? c : c * inv_alpha;
          if (l.ckpt && valid) h = l.ckpt[(int64_t)row * l.d_out + n];   // (re-seed)
          const int at = row * pitch + place(n);
          X[xo * size + at] = valid ? (fresh ? z : l.alpha * z) : 0.f;
          C[ci * size + at] = valid ? c : 0.f;
          H[(1 - hi) * size + at] = valid ? h : 0.f;
        }
      }
    }
    if (i > 0) {
      const SmallLayer& l = p.layer[i - 1];
      const int mt = l.out.tiles, nt = l.in.tiles;
      const float* const ct = C + (1 - ci) * size;
      const float* const x = X + (xi == 0 ? 2 : xi - 1) * size;
      int mm = (int)(l.out.at >> (4 * wave) & 15u) * 16, nn = (int)(l.out.round >> (4 * wave) & 15u) * 16;
      while (nn < nt * 16) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < p.rows; s += 32) {
          float fa[8], fb[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int k = s + 16 * (q & 1) + (q >> 1) + 2 * u;
            fa[u] = ct[k * pitch + place(mm + r)];
            fb[u] = x[k * pitch + place(nn + r)];
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[u], fb[u], acc, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int row = mm + 4 * q + j, col = nn + r;
          if (row >= l.d_out || col >= l.d_in) continue;
          float* const dst = l.dW + (int64_t)row * l.d_in + col;
          float v = p.scale * acc[j];
          if (p.beta != 0.f) v += p.beta * *dst;
          *dst = v;
        }
        for (mm += 16 * WAVES; mm >= 16 * mt; mm -= 16 * mt) nn += 16;   // eight tiles on
      }
      // column sums: the lower and the upper sixteen of every 32 rows, then the two
      if (l.db && threadIdx.x < 2 * SMALL_NET_MAX_WIDTH) {
        const int c = threadIdx.x >> 1, half = threadIdx.x & 1;
        float sum = 0.f;
        if (c < l.d_out)
          for (int s = 0; s < p.rows; s += 32)
#pragma unroll
            for (int k = 0; k < 16; ++k) sum += ct[(s + 16 * half + k) * pitch + place(c)];
        const float both = sum + __shfl_xor(sum, 1);
        if (c < l.d_out && half == 0) {
          float v = p.scale * both;
          if (p.beta != 0.f) v += p.beta * l.db[c];
          l.db[c] = v;
        }
      }
    }
    if (i < L) {
      w = next;
      pw = next_pw;
      __syncthreads();
      xi = xi == 2 ? 0 : xi + 1;
      hi = 1 - hi;
      ci = 1 - ci;
    }
  }
  if (mism) atomicAdd(reinterpret_cast<unsigned long long*>(p.status), (unsigned long long)mism);
}

}  // namespace

hipError_t small_net_step(const SmallNet& n, hipStream_t stream) {
  static hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void*>(k_small_net), hipFuncAttributeMaxDynamicSharedMemorySize, SMALL_NET_MAX_LDS);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(k_small_net, dim3(1), dim3(NT), (size_t)(7 * n.rows * n.pitch + n.bit_words) * sizeof(float), stream, n);
  return hipGetLastError();
}

}  // namespace mw
