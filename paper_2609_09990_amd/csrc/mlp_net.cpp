// The preconditioner network on the GPU: parameters, forward (fp32 or bf16
// hidden layer on the matrix cores), cosine loss with backward, and Adam.
#include <algorithm>
#include <cmath>

#include "mlp.hpp"

namespace dmrg {

namespace {
struct SplitMix {
  uint64_t s;
  uint64_t next() {
    uint64_t z = (s += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
  }
  double normal() {
    double u1 = ((next() >> 11) + 0.5) * (1.0 / 9007199254740992.0);
    double u2 = ((next() >> 11) + 0.5) * (1.0 / 9007199254740992.0);
    return std::sqrt(-2.0 * std::log(u1)) * std::cos(6.283185307179586 * u2);
  }
};
}  // namespace

MLP::MLP(int n_in, int width, unsigned long long seed, hipStream_t s) : nin_(n_in), w_(width), st_(s) {
  DMRG_REQUIRE(n_in >= 1 && n_in <= 64 && width >= 1 && width <= 1024, ST_EINVAL, "network shape out of range");
  oW1_ = 0;
  ob1_ = oW1_ + (long)w_ * nin_;
  oW2_ = ob1_ + w_;
  ob2_ = oW2_ + (long)w_ * w_;
  oW3_ = ob2_ + w_;
  ob3_ = oW3_ + w_;
  np_ = ob3_ + 1;
  // He-normal weights, zero biases
  std::vector<float> h(np_, 0.f);
  SplitMix rng{seed};
  for (long i = 0; i < (long)w_ * nin_; ++i) h[oW1_ + i] = (float)(rng.normal() * std::sqrt(2.0 / nin_));
  for (long i = 0; i < (long)w_ * w_; ++i) h[oW2_ + i] = (float)(rng.normal() * std::sqrt(2.0 / w_));
  for (long i = 0; i < w_; ++i) h[oW3_ + i] = (float)(rng.normal() * std::sqrt(1.0 / w_));
  p_.reserve(np_ * 4);
  m_.reserve(np_ * 4);
  v_.reserve(np_ * 4);
  grad_.reserve(np_ * 4);
  w2b_.reserve((size_t)w_ * w_ * 2);
  set_params(h.data());
}

void MLP::refresh_bf16() { launch_f32_to_bf16_rne(p_.as<float>() + oW2_, w2b_.as<uint16_t>(), (long)w_ * w_, st_); }

void MLP::set_params(const float* host) {
  hip_check(hipMemcpyAsync(p_.p, host, np_ * 4, hipMemcpyHostToDevice, st_), "mlp params");
  hip_check(hipMemsetAsync(m_.p, 0, np_ * 4, st_), "adam m");
  hip_check(hipMemsetAsync(v_.p, 0, np_ * 4, st_), "adam v");
  hip_check(hipMemsetAsync(grad_.p, 0, np_ * 4, st_), "grad");
  t_ = 0;
  refresh_bf16();
  hip_check(hipStreamSynchronize(st_), "mlp params");
}

void MLP::get_params(float* host) const {
  hip_check(hipMemcpyAsync(host, p_.p, np_ * 4, hipMemcpyDeviceToHost, st_), "mlp params");
  hip_check(hipStreamSynchronize(st_), "mlp params");
}

// C[rows x W] = A[rows x W] W2^T (operands of `prec`) on 64 x 64 tiles: one item
// per 64-row tile (the A operand moves with the tile), all W columns.
void MLP::gemm(Tables& t, int prec, const void* A, const void* B, void* C, long rows, hipStream_t s) {
  if (t.key[0] != A || t.key[1] != B || t.key[2] != C || t.rows != rows) {
    hip_check(hipStreamSynchronize(s), "mlp tables");  // earlier uploads of the staging vectors are done
    t.rows = -1;  // no tables until these are uploaded
    t.hu.clear();
    t.hi.clear();
    for (long m0 = 0; m0 < rows; m0 += 64) {
      int ib = (int)t.hi.size();
      t.hi.push_back({(const char*)A + m0 * w_ * (prec == PREC_BF16 ? 2 : 4), B, w_, w_, w_, 0, 1.0});
      char* Cm = (char*)C + m0 * w_ * 4;
      const int M = (int)std::min<long>(64, rows - m0);
      for (int n0 = 0; n0 < w_; n0 += 64) t.hu.push_back({Cm, w_, M, w_, 0, n0, ib, ib + 1, 0});
    }
    t.du.reserve(t.hu.size() * sizeof(GemmUnit) + 64);
    t.di.reserve(t.hi.size() * sizeof(GemmItem) + 64);
    hip_check(hipMemcpyAsync(t.du.p, t.hu.data(), t.hu.size() * sizeof(GemmUnit), hipMemcpyHostToDevice, s), "mlp units");
    hip_check(hipMemcpyAsync(t.di.p, t.hi.data(), t.hi.size() * sizeof(GemmItem), hipMemcpyHostToDevice, s), "mlp items");
    t.key[0] = A;
    t.key[1] = B;
    t.key[2] = C;
    t.rows = rows;
    t.nu = (int)t.hu.size();
  }
  launch_gemm(prec, GEMM_NT, t.du.as<GemmUnit>(), t.nu, t.di.as<GemmItem>(), s);
}

void MLP::forward(int prec, const float* X, long n, float* y, hipStream_t s) {
  DMRG_REQUIRE(prec == PREC_F32 || prec == PREC_BF16, ST_EINVAL, "network precision must be FP32 or BF16");
  if (n <= 0) return;
  if (!s) s = st_;
  const float* P = p_.as<float>();
  if (prec == PREC_BF16 && launch_mlp_infer_bf16(X, n, nin_, P + oW1_, P + ob1_, w_, w2b_.as<uint16_t>(), P + ob2_,
                                                 P + oW3_, P + ob3_, y, s))
    return;
  if (prec == PREC_BF16) {
    z2_.reserve((size_t)n * w_ * 4);
    a1b_.reserve((size_t)n * w_ * 2);
    launch_mlp_layer1(X, n, nin_, P + oW1_, P + ob1_, w_, nullptr, a1b_.as<uint16_t>(), s);
    gemm(ti_, PREC_BF16, a1b_.p, w2b_.p, z2_.p, n, s);
    launch_mlp_layer3(z2_.as<float>(), n, w_, P + ob2_, P + oW3_, P + ob3_, y, false, s);
    return;
  }
  forward_f32(X, n, y, false, s);
}

void MLP::forward_f32(const float* X, long n, float* y, bool keep, hipStream_t s) {
  const float* P = p_.as<float>();
  const bool few = mlp_few_tiles(n, w_);
  a1_.reserve((size_t)n * w_ * 4);
  if (few || keep) z2_.reserve((size_t)n * w_ * 4);
  if (!few) part_.reserve((size_t)mlp_layer3_parts(w_) * n * 8);
  launch_mlp_layer1(X, n, nin_, P + oW1_, P + ob1_, w_, a1_.as<float>(), nullptr, s);
  if (few) {
    gemm(tz_, PREC_F32, a1_.p, P + oW2_, z2_.p, n, s);
    launch_mlp_layer3(z2_.as<float>(), n, w_, P + ob2_, P + oW3_, P + ob3_, y, keep, s);
  } else {
    launch_mlp_forward_f32(a1_.as<float>(), n, w_, P + oW2_, P + ob2_, P + oW3_, P + ob3_,
                           keep ? z2_.as<float>() : nullptr, part_.as<double>(), y, s);
  }
}

double MLP::loss_grad(const float* X, const float* T, int nseg, int seglen) {
  DMRG_REQUIRE(nseg >= 1 && seglen >= 1, ST_EINVAL, "empty training batch");
  const long n = (long)nseg * seglen;
  const float* P = p_.as<float>();
  float* G = grad_.as<float>();
  y_.reserve((size_t)n * 4);
  dy_.reserve((size_t)n * 4);
  stats_.reserve((size_t)nseg * 3 * 8);
  const long nch = mlp_row_chunks(n), nrt = mlp_row_tiles(n);
  part_.reserve((size_t)std::max((long)mlp_layer3_parts(w_) * n, std::max(2 * nch, (nin_ + 1) * nrt) * w_) * 8);
  gpart_.reserve((size_t)nch * w_ * w_ * 4);
  // forward (fp32), keeping a1 and a2 (z2_ holds a2)
  forward_f32(X, n, y_.as<float>(), true, st_);
  // loss and dL/dy
  launch_seg_stats(y_.as<float>(), T, nseg, seglen, stats_.as<double>(), st_);
  launch_cos_grad(y_.as<float>(), T, stats_.as<double>(), nseg, seglen, dy_.as<float>(), st_);
  // db3 = sum_i dy_i, then everything below it
  launch_sum_all(dy_.as<float>(), n, part_.as<double>(), G + ob3_, st_);
  launch_mlp_backward_f32(X, nin_, a1_.as<float>(), z2_.as<float>(), dy_.as<float>(), n, w_, P + oW2_, P + oW3_,
                          part_.as<double>(), gpart_.as<float>(), G + oW1_, G + ob1_, G + oW2_, G + ob2_, G + oW3_,
                          st_);
  std::vector<double> hs((size_t)nseg * 3);
  hip_check(hipMemcpyAsync(hs.data(), stats_.p, hs.size() * 8, hipMemcpyDeviceToHost, st_), "loss");
  hip_check(hipStreamSynchronize(st_), "loss");
  double loss = 0.0;
  for (int s = 0; s < nseg; ++s) {
    double yt = hs[3 * s], yy = hs[3 * s + 1], tt = hs[3 * s + 2];
    double c = (yy > 0 && tt > 0) ? yt / std::sqrt(yy * tt) : 0.0;
    loss += (1.0 - c) / nseg;
  }
  return loss;
}

void MLP::adam(float lr, float beta1, float beta2, float eps) {
  ++t_;
  const float c1 = 1.f - std::pow(beta1, (float)t_), c2 = 1.f - std::pow(beta2, (float)t_);
  launch_adam(p_.as<float>(), m_.as<float>(), v_.as<float>(), grad_.as<float>(), np_, lr, beta1, beta2, eps, c1, c2,
              st_);
  refresh_bf16();
  hip_check(hipStreamSynchronize(st_), "adam");
}

}  // namespace dmrg
