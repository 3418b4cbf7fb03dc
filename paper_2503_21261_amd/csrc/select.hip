// Squared quantisation error of the rotated g_y under per-token and per-tensor
// scales: the measurement behind Layer-wise Quantizer Selection (Sec. 5.2.2).
// Calibration-time only; sums are double and combined in a fixed order so the
// result is reproducible run to run.
//
// Two passes over g_y, rows held in registers as in row_quant_kernel.h: the first finds each row's
// abs-max and sums the per-token error on the spot, the second sums the per-tensor error.  A third
// kernel adds the workgroups' sums.  HBM-bound in the first pass at about the arithmetic's own
// rate (per element and pass: the butterflies, ten instructions of quantisation and four fp64 ones:
// the product of code and scale is exact in fp64, so it goes into a fused multiply-add).
// 16384 x 4096, 64-element blocks: 58 + 49 + 6 us (4.6 and 5.5 TB/s); with one error pass for both
// scales, a separate multiply and two instructions per stage across lanes it was 49 + 88 + 20 us.
#include "hot_host.h"
#include "row_quant_kernel.h"

namespace hot {

// The quantiser's code as a float (quant_code's value), the random fraction m / 2048 as the
// difference of two floats of which 1/2048 is the unit in the last place.
template <int ROUNDING>
__device__ __forceinline__ float quant_code_float(float t, float inv, float qmax) {
  const float v = t * inv;
  float q;
  if constexpr (ROUNDING == 0) {
    q = rintf(v);
  } else {
    const float f = floorf(v);
    const float rnd = __uint_as_float(0x45800000u | (__float_as_uint(v) & 0x7FFu)) - 4096.0f;
    q = v - f > rnd ? f + 1.0f : f;
  }
  return fminf(fmaxf(q, -qmax), qmax);
}

// sum + the squared errors (t - q(t) * scale)^2 of four elements.  inv and scale carry the sign the
// lane's values are held with.
template <int ROUNDING>
__device__ __forceinline__ double add_sq_err4(double sum, const float4& t, float inv, double scale, float qmax) {
  const float e[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double d = fma(-(double)quant_code_float<ROUNDING>(e[i], inv, qmax), scale, (double)e[i]);
    sum = fma(d, d, sum);
  }
  return sum;
}

// The same under a scale whose inverse is infinite (abs-max below qmax / FLT_MAX, 2e-38 for INT4): the
// quantiser's product is infinite, or, for a zero, a NaN that its conversion to an integer makes 0.
// Rare; the opaque copies keep the usual case's registers free of what the compiler would share.
__device__ __forceinline__ double add_saturated_sq_err4(double sum, const float4& t, float inv, double scale, float qmax) {
  float e[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    asm volatile("" : "+v"(e[i]));
    const float q = e[i] == 0.0f ? 0.0f : copysignf(qmax, e[i] * inv);
    const double d = fma(-(double)q, scale, (double)e[i]);
    sum = fma(d, d, sum);
  }
  return sum;
}

struct SelectArgs {
  const float* t;
  int64_t rows;
  int cols, bits, rounding;
  float* partials;   // per-token pass: out, the workgroups' maxima; per-tensor pass: in
  int npartials;
  double* sums;      // [workgroup of the pass]
};

// End of a pass: the workgroup's error sum and (per-token pass) abs-max.
template <bool TOKEN, int WAVES = 4>
__device__ __forceinline__ void leave_sums(const SelectArgs& a, double sum, float running) {
  __shared__ double s_sum[WAVES];
  __shared__ float s_run[WAVES];
  const int tid = threadIdx.x;
#pragma unroll
  for (int m = 1; m < 64; m *= 2) sum += __shfl_xor(sum, m);
  if constexpr (TOKEN) running = wave_max(running);
  if ((tid & 63) == 0) { s_sum[tid >> 6] = sum; s_run[tid >> 6] = running; }
  __syncthreads();
  if (tid == 0) {
    double total = 0.0;
    float most = 0.0f;
#pragma unroll
    for (int w = 0; w < WAVES; w += 4) {
      total += (s_sum[w] + s_sum[w + 1]) + (s_sum[w + 2] + s_sum[w + 3]);
      most = fmaxf(most, fmaxf(fmaxf(s_run[w], s_run[w + 1]), fmaxf(s_run[w + 2], s_run[w + 3])));
    }
    a.sums[blockIdx.x] = total;
    if constexpr (TOKEN) a.partials[blockIdx.x] = most;
  }
}

template <int N, int ITER, int TPR, bool TOKEN>
__global__ __launch_bounds__(256) void select_rows_kernel(const SelectArgs a) {
  constexpr int RPB = 256 / TPR;
  __shared__ float s_max[4];
  const int tid = threadIdx.x, rl = tid / TPR;
  const RowLane<N> lane = row_lane<N>(tid % TPR);
  const int tr = lane.id;
  const int qmax = (1 << (a.bits - 1)) - 1;
  const int64_t nrb = (a.rows + RPB - 1) / RPB;
  float amax = 0.0f, running = 0.0f;
  if constexpr (!TOKEN) amax = block_max_of(a.partials, a.npartials);
  double sum = 0.0;
  for (int64_t rb0 = blockIdx.x; rb0 < nrb; rb0 += gridDim.x) {
    // the second pass starts where the first one ended (what the memory-side cache still holds)
    const int64_t row = (TOKEN ? rb0 : nrb - 1 - rb0) * RPB + rl;
    const bool row_ok = row < a.rows;
    const float4* src = reinterpret_cast<const float4*>(a.t + row * (int64_t)a.cols);
    float4 v[ITER];
    float m = 0.0f;
#pragma unroll
    for (int it = 0; it < ITER; ++it)
      v[it] = (row_ok && (it * TPR + tr) * 4 < a.cols) ? src[it * TPR + tr] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      fwht_row4<N>(v[it], lane);
      m = fmaxf(m, absmax4(v[it]));
    }
    if constexpr (TOKEN) {
      amax = row_max<TPR>(m, s_max);
      running = fmaxf(running, amax);
    }
    const float inv = flip_sign(quant_inv(amax, qmax), lane.flip);
    const double scale = (double)flip_sign(quant_scale(amax, qmax), lane.flip);
    if (isinf(inv)) {   // elements past the row's end are zeros with zero error, here as below
#pragma unroll
      for (int it = 0; it < ITER; ++it) sum = add_saturated_sq_err4(sum, v[it], inv, scale, (float)qmax);
    } else if (a.rounding == 0) {
#pragma unroll
      for (int it = 0; it < ITER; ++it) sum = add_sq_err4<0>(sum, v[it], inv, scale, (float)qmax);
    } else {
#pragma unroll
      for (int it = 0; it < ITER; ++it) sum = add_sq_err4<1>(sum, v[it], inv, scale, (float)qmax);
    }
  }
  leave_sums<TOKEN>(a, sum, running);
}

// Rows a part at a time, one per workgroup: those too long for 256 threads' registers, in the per-token
// pass with the first kStreamHeld float4 of a thread kept and only what lies beyond read twice; and
// the per-tensor pass, which has no use for a whole row, of the longest that registers hold (few of
// their workgroups fit a unit).  4096 rows of 11392: 129 us with whole rows in both passes, 110 so; of
// 16448 with nothing kept 164, 148 so.
constexpr int kStreamHeld = 8;
template <int N, bool TOKEN, int NT>
__global__ __launch_bounds__(NT) void select_stream_kernel(const SelectArgs a) {
  __shared__ float s_max[NT / 64];
  const int tid = threadIdx.x;
  const int qmax = (1 << (a.bits - 1)) - 1;
  const RowLane<N> lane = row_lane<N>(tid);
  const int nvec = a.cols / 4;
  float amax = 0.0f, running = 0.0f;
  if constexpr (!TOKEN) amax = block_max_of(a.partials, a.npartials);
  double sum = 0.0;
  for (int64_t r = blockIdx.x; r < a.rows; r += gridDim.x) {
    const int64_t row = TOKEN ? r : a.rows - 1 - r;   // as in select_rows_kernel
    const float4* src = reinterpret_cast<const float4*>(a.t + row * (int64_t)a.cols);
    auto transformed = [&](int base) {   // uniform trip counts keep the lanes of a butterfly together
      float4 q = base + lane.id < nvec ? src[base + lane.id] : make_float4(0.f, 0.f, 0.f, 0.f);
      fwht_row4<N>(q, lane);
      return q;
    };
    constexpr int HELD = TOKEN ? kStreamHeld : 0;
    float4 held[HELD > 0 ? HELD : 1];
    if constexpr (TOKEN) {
      float m = 0.0f;
#pragma unroll
      for (int it = 0; it < HELD; ++it) {
        const int i = it * NT + lane.id;
        held[it] = i < nvec ? src[i] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int it = 0; it < HELD; ++it) {
        fwht_row4<N>(held[it], lane);
        m = fmaxf(m, absmax4(held[it]));
      }
      for (int base = NT * HELD; base < nvec; base += NT) m = fmaxf(m, absmax4(transformed(base)));
      m = wave_max(m);
      if ((tid & 63) == 0) s_max[tid >> 6] = m;
      __syncthreads();
      amax = 0.0f;
#pragma unroll
      for (int w = 0; w < NT / 64; ++w) amax = fmaxf(amax, s_max[w]);
      __syncthreads();
      running = fmaxf(running, amax);
    }
    const float inv = flip_sign(quant_inv(amax, qmax), lane.flip);
    const double scale = (double)flip_sign(quant_scale(amax, qmax), lane.flip);
    if (isinf(inv)) {
      for (int base = 0; base < nvec; base += NT)
        sum = add_saturated_sq_err4(sum, transformed(base), inv, scale, (float)qmax);
      continue;
    }
#pragma unroll
    for (int it = 0; it < HELD; ++it)
      sum = a.rounding == 0 ? add_sq_err4<0>(sum, held[it], inv, scale, (float)qmax)
                            : add_sq_err4<1>(sum, held[it], inv, scale, (float)qmax);
    for (int base = NT * HELD; base < nvec; base += NT) {
      const float4 q = transformed(base);
      sum = a.rounding == 0 ? add_sq_err4<0>(sum, q, inv, scale, (float)qmax)
                            : add_sq_err4<1>(sum, q, inv, scale, (float)qmax);
    }
  }
  leave_sums<TOKEN, NT / 64>(a, sum, running);
}

// Single workgroup: result[c] = sum of sums[c][0 .. count), fixed order.
__global__ __launch_bounds__(256) void select_final_kernel(const double* __restrict__ sums, int count,
                                                           double* __restrict__ result) {
  __shared__ double s_sum[2][256];
  const int tid = threadIdx.x;
  double a = 0.0, b = 0.0;
  for (int i = tid; i < count; i += 256) { a += sums[i]; b += sums[count + i]; }
  s_sum[0][tid] = a;
  s_sum[1][tid] = b;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) { s_sum[0][tid] += s_sum[0][tid + h]; s_sum[1][tid] += s_sum[1][tid + h]; }
    __syncthreads();
  }
  if (tid == 0) { result[0] = s_sum[0][0]; result[1] = s_sum[1][0]; }
}

namespace {

// Float4 per thread from which the per-tensor pass streams its rows (4096 rows of 9216: 97 us held, 90
// streamed; at 6, 1024 rows of 6144, 46 either way).
constexpr int kStreamFrom = 8;
// Longest streamed rows whose first pass runs on 256 threads (4096 rows of 20480: 175 us, 185 on 1024
// threads; of 32768 276 and 240).
constexpr int kFewThreads = 20480;

template <int N>
hipError_t launch_passes(SelectArgs a, double* result, hipStream_t s) {
  double* const sums = a.sums;
  unsigned grid = 0;
  const bool held = with_row_layout(a.cols, [&](auto iter_c, auto tpr_c) {
    constexpr int ITER = decltype(iter_c)::value, TPR = decltype(tpr_c)::value;
    const int64_t nrb = ceil_div(a.rows, 256 / TPR);
    grid = (unsigned)(nrb < kMaxPartials ? nrb : kMaxPartials);
    a.npartials = (int)grid;
    select_rows_kernel<N, ITER, TPR, true><<<dim3(grid), dim3(256), 0, s>>>(a);
    a.sums = sums + grid;
    if constexpr (ITER >= kStreamFrom) select_stream_kernel<N, false, 256><<<dim3(grid), dim3(256), 0, s>>>(a);
    else select_rows_kernel<N, ITER, TPR, false><<<dim3(grid), dim3(256), 0, s>>>(a);
  });
  if (!held) {
    grid = (unsigned)(a.rows < kMaxPartials ? a.rows : kMaxPartials);
    a.npartials = (int)grid;
    if (a.cols <= kFewThreads) select_stream_kernel<N, true, 256><<<dim3(grid), dim3(256), 0, s>>>(a);
    else select_stream_kernel<N, true, 1024><<<dim3(grid), dim3(1024), 0, s>>>(a);
    a.sums = sums + grid;
    select_stream_kernel<N, false, 256><<<dim3(grid), dim3(256), 0, s>>>(a);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  select_final_kernel<<<dim3(1), dim3(256), 0, s>>>(sums, (int)grid, result);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_select(const float* t, int64_t rows, int64_t cols, int n, int bits, int rounding,
                         float* partials, double* sums, double* result, hipStream_t s) {
  const SelectArgs a{t, rows, (int)cols, bits, rounding, partials, 0, sums};
  switch (n) {
    case 16: return launch_passes<16>(a, result, s);
    case 32: return launch_passes<32>(a, result, s);
    case 64: return launch_passes<64>(a, result, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace hot
