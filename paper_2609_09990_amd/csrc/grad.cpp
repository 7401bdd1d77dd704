// Gradient of the MPS energy with respect to the active-space integrals: the
// Hellmann-Feynman contribution of the DMRG node's adjoint (Sec. II.C, the
// sweep as a differentiable node; Eq. (implicit) needs no response solve for
// the energy of a simple root of a stationary state).  The MPS is held fixed,
// so dE/dh and dE/dB^Q are contractions of the state's one- and two-body
// densities; those densities are never formed here.
//
// <Psi|H|Psi> is linear in the coefficients of the entries of any one MPO site.
// For an entry e = (alpha -> beta, c op) of W_k,
//   g_e = d<Psi|H|Psi>/dc_e = sum_{s s'} op[s][s'] < A_s R_{k+1}[beta] , L_k[alpha] A_s' >_F
// with the environments L_k (sites < k) and R_{k+1} (sites > k) of the stored
// MPS (any gauge).  The vectors P_{alpha,s'} = L_k[alpha] A_s' and
// Q_{beta,s} = A_s R_{k+1}[beta] live on blocks (i, j') of bond k x bond k+1
// with q(j') - q(i) fixed per (channel, state); grouped by that offset, every
// needed inner product is an entry of a dense G = P Q^T, a long-K GEMM on the
// fp64 matrix cores.  The MPO builder's provenance (d coefficient / d
// parameter) maps g to dE/dh_pq, dE/d(pq|rs) and dE/dB^Q_pq, and
// (pq|rs) = sum_Q B^Q_pq B^Q_rs carries the middle one back to B.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <map>

#include "solver.hpp"

namespace dmrg {

namespace {

struct PairBlock {
  int i, j;   // bond-k sector (bra), bond-(k+1) sector (ket)
  int mi, mj;
  long off;
};

struct PairClass {
  QN delta;  // q(j) - q(i)
  std::vector<PairBlock> blocks;
  long K = 0;
  std::vector<std::pair<int, int>> prow, qrow;  // (alpha, s'), (beta, s)
  std::vector<int> prow_of, qrow_of;
};

// Host tables of one side's rows, packed for one upload (launch_grad_expand).
struct GradPlan {
  std::vector<GradJob> jobs;
  std::vector<GradTile> tiles;
  std::vector<GradBlock> blocks;
  std::vector<GradSrc> srcs;
  std::vector<GradRow> rows;
  std::vector<char> packed;
  long units = 0;
  double flops = 0;
  bool buf = true;  // every product fits the buffer-load kernels
  void clear() { *this = GradPlan(); }
  template <class T>
  size_t put(const std::vector<T>& v) {
    const size_t at = (packed.size() + 15) / 16 * 16;
    packed.resize(at + v.size() * sizeof(T));
    if (!v.empty()) std::copy((const char*)v.data(), (const char*)(v.data() + v.size()), packed.data() + at);
    return at;
  }
  size_t at[5] = {0, 0, 0, 0, 0};
  void pack() {
    at[0] = put(jobs);
    at[1] = put(tiles);
    at[2] = put(blocks);
    at[3] = put(srcs);
    at[4] = put(rows);
  }
  GradView view(const char* d) const {
    return {(const GradJob*)(d + at[0]), (const GradTile*)(d + at[1]), (const GradBlock*)(d + at[2]),
            (const GradSrc*)(d + at[3]), (const GradRow*)(d + at[4]), (int)jobs.size(), units};
  }
};

// Index of row (channel ch, state s), added on first use; idx: (channel, state) -> row.
int row_index(std::vector<std::pair<int, int>>& rows, std::vector<int>& idx, int ch, int s) {
  const size_t at = 4 * (size_t)ch + s;
  if (at >= idx.size()) idx.resize(at + 1, -1);
  if (idx[at] < 0) {
    idx[at] = (int)rows.size();
    rows.push_back({ch, s});
  }
  return idx[at];
}

// Largest P or Q chunk of one class, in doubles (two such buffers are live at once).
constexpr long kChunkElems = 1L << 29;
// Classes run together while their P and their Q rows stay below this many doubles
// (CAS(16,16), M = 256: 54 ms with 2^26 and with 2^29, 59 with 2^24).
constexpr long kBatchElems = 1L << 26;
// P, Q and G buffers kept between calls, in bytes.
constexpr size_t kKeepBytes = size_t(1) << 30;
// K extent of one item of the G = P Q^T product (split-K granule).
constexpr int kGSplit = 4096;

}  // namespace

size_t GradWork::bytes() const {
  size_t n = P.bytes + Q.bytes + G.bytes;
  for (const Tables& t : tab) n += t.tables.bytes + t.units.bytes + t.items.bytes;
  for (int i = 0; i < 3; ++i) n += ph.d_items[i].bytes + ph.d_units[i].bytes + ph.d_tiles[i].bytes;
  return n;
}

void GradWork::release() {
  P.release();
  Q.release();
  G.release();
  for (Tables& t : tab) t = Tables();
  ph = Phase();
}

void GradWork::drop() {
  std::lock_guard<std::mutex> l(m_);
  if (users_ == 0 && !arena_) release();
}

void GradWork::enter(int d) {
  std::lock_guard<std::mutex> l(m_);
  users_ += d;
  if (d > 0) arena_ = current_arena() != nullptr;
}

// g[e] = d<Psi|H|Psi>/dc_e for every entry of W_k (unnormalised state); with
// norm != nullptr also <Psi|Psi> = sum_s < A_s R_{k+1}[H], L_k[I] A_s >_F (the
// channels that are the identity on the left and on the right block).
void Solver::grad_site(int k, std::vector<double>& g, double* norm) {
  const MPO& mpo = prob_->mpo;
  GradWork::Use use(grad_);
  try {
    ensure_left(k);
    ensure_right(k + 1);
  } catch (const Error& e) {  // again without the buffers of the site before
    if (e.code != ST_ENOMEM || grad_.bytes() == 0) throw;
    hip_check(hipStreamSynchronize(st), "grad site");
    grad_.release();
    ensure_left(k);
    ensure_right(k + 1);
  }
  const Env& envl = left_[k];
  const Env& envr = right_[k + 1];
  const Bond& bl = bonds_[k];
  const Bond& br = bonds_[k + 1];
  const SiteTensor& A = mps_[k];
  const auto& W = mpo.W[k];
  g.assign(W.size(), 0.0);

  // classes of (i, j') blocks by quantum-number offset; rows each entry needs
  std::vector<PairClass> classes;
  auto get_class = [&](QN d) {
    for (size_t c = 0; c < classes.size(); ++c)
      if (classes[c].delta == d) return (int)c;
    PairClass pc;
    pc.delta = d;
    for (int i = 0; i < (int)bl.sec.size(); ++i) {
      int j = br.find(bl.sec[i].q + d);
      if (j < 0) continue;
      pc.blocks.push_back({i, j, bl.sec[i].dim, br.sec[j].dim, pc.K});
      pc.K += (long)bl.sec[i].dim * br.sec[j].dim;
    }
    int c = (int)classes.size();
    classes.push_back(std::move(pc));
    return c;
  };
  struct Use { int cls, pr, qr; double w; };
  std::vector<std::vector<Use>> uses(W.size());
  const auto& chl = mpo.chans[k];
  const auto& chr = mpo.chans[k + 1];
  for (size_t e = 0; e < W.size(); ++e) {
    const Mat4& op = mpo.ops[W[e].op];
    for (int s = 0; s < 4; ++s)
      for (int sp = 0; sp < 4; ++sp) {
        double w = op[s * 4 + sp];
        if (w == 0.0) continue;
        QN d = site_qn(sp) - chl[W[e].a].dq;
        DMRG_REQUIRE(d == site_qn(s) - chr[W[e].b].dq, ST_EINVAL, "MPO entry breaks quantum-number conservation");
        int c = get_class(d);
        if (classes[c].K == 0) continue;
        int pr = row_index(classes[c].prow, classes[c].prow_of, W[e].a, sp);
        int qr = row_index(classes[c].qrow, classes[c].qrow_of, W[e].b, s);
        uses[e].push_back({c, pr, qr, w});
      }
  }
  std::vector<Use> norm_uses;
  if (norm) {
    const int I = mpo.chan_I[k], H = mpo.chan_H[k + 1];
    DMRG_REQUIRE(I >= 0 && H >= 0, ST_EINVAL, "no identity channels for the norm at this site");
    for (int s = 0; s < 4; ++s) {
      QN d = site_qn(s) - chl[I].dq;
      DMRG_REQUIRE(d == site_qn(s) - chr[H].dq, ST_EINVAL, "identity channels with a charge");
      int c = get_class(d);
      if (classes[c].K == 0) continue;
      int pr = row_index(classes[c].prow, classes[c].prow_of, I, s);
      int qr = row_index(classes[c].qrow, classes[c].qrow_of, H, s);
      norm_uses.push_back({c, pr, qr, 1.0});
    }
    *norm = 0.0;
  }

  // Products of several classes run together (one launch each for all their P
  // rows, Q rows and G = P Q^T, one read-back): a site's classes are many and
  // small, and taken one at a time each cost three plans, six launches and a
  // synchronisation (243 of them at CAS(12,12), M = 256).  Together they take
  // at most kBatchElems or, beyond it, what the largest of them takes alone.
  // A class whose rows exceed the chunk bound runs by itself in chunks of rows.
  struct Job {
    size_t c;
    int p0, np, q0, nq;
    long poff, qoff, goff;  // elements of this job's P, Q, G in the buffers
    bool fresh_p;           // P rows to be formed (not those of the job before)
  };
  std::vector<std::vector<double>> Gc(classes.size());
  std::vector<Job> batch;
  long bp = 0, bq = 0, bg = 0;
  std::vector<double> Ghost;
  // The P and Q rows' products (row r, block (i, j'), tile) are made on the device
  // from tables of the rows and of the blocks: P_{alpha,s'}[i, j'] = L_k[alpha](i, i')
  // A(i', s', j') and Q_{beta,s}[i, j'] = A(i, s, j) R_{k+1}[beta](j, j').  A row's
  // channel class fixes its state and sectors, so the tables are (classes) x
  // (blocks), not (rows) x (blocks); a block without a source is written as zeros.
  auto make_rows = [&](bool left, GradPlan& gp) {
    const Env& env = left ? envl : envr;
    const auto& chans = left ? chl : chr;
    gp.clear();
    for (const Job& jb : batch) {
      const PairClass& pc = classes[jb.c];
      const int nr = left ? jb.np : jb.nq, r0 = left ? jb.p0 : jb.q0;
      if (nr == 0 || (left && !jb.fresh_p)) continue;
      GradJob J{};
      J.u0 = gp.units;
      J.out = left ? jb.poff : jb.qoff;
      J.K = pc.K;
      J.tile0 = (int)gp.tiles.size();
      J.blk0 = (int)gp.blocks.size();
      J.src0 = (int)gp.srcs.size();
      J.row0 = (int)gp.rows.size();
      J.nblk = (int)pc.blocks.size();
      for (int i = 0; i < J.nblk; ++i) {
        const PairBlock& pb = pc.blocks[i];
        gp.blocks.push_back({pb.off, pb.mi, pb.mj});
        for (int m0 = 0; m0 < pb.mi; m0 += 64)
          for (int n0 = 0; n0 < pb.mj; n0 += 32)
            gp.tiles.push_back({i, m0, n0, 8 * ((std::min(64, pb.mi - m0) + 15) / 16) + (std::min(32, pb.mj - n0) + 15) / 16});
      }
      J.ntile = (int)gp.tiles.size() - J.tile0;
      std::vector<int> kind_of(env.classes.size(), -1);
      int kinds = 0;
      for (int r = 0; r < nr; ++r) {
        const auto& row = left ? pc.prow[r0 + r] : pc.qrow[r0 + r];
        const int ch = row.first, st_idx = row.second, cls = env.chan_class[ch];
        const EnvClass& ec = env.classes[cls];
        if (kind_of[cls] < 0) {
          kind_of[cls] = kinds++;
          for (const PairBlock& pb : pc.blocks) {
            GradSrc x{0, 0, 0, 0, 0, 0};
            // sectors of the site block: (ip, s', j') on the left, (i, s, j) on the right
            const int ip = left ? bl.find(bl.sec[pb.i].q - chans[ch].dq) : pb.i;
            const int j = left ? pb.j : br.find(bl.sec[pb.i].q + site_qn(st_idx));
            const int sl = ip < 0 || j < 0 ? -1 : A.lay.slab_of_left[ip];
            const int ab = sl < 0 ? -1 : A.lay.slabs[sl].block_of(st_idx, j);
            const int eb = ab < 0 ? -1 : ec.block_of_col[left ? ip : pb.j];
            if (eb >= 0 && ec.blocks[eb].ri == (left ? pb.i : j)) {
              const Slab& slab = A.lay.slabs[sl];
              x.env = ec.blocks[eb].off;
              x.site = slab.off + slab.blocks[ab].col0;
              x.K = left ? ec.blocks[eb].mc : br.sec[j].dim;
              x.lda = left ? ec.blocks[eb].mc : slab.width;
              x.ldb = left ? slab.width : ec.blocks[eb].mc;
              x.valid = 1;
              // host check of what the products read, for this class's last channel
              const long ea = (long)(pb.mi - 1) * x.lda + x.K, eb2 = (long)(x.K - 1) * x.ldb + pb.mj;
              DMRG_REQUIRE(x.env + (left ? ea : eb2) <= ec.nnz && x.site + (left ? eb2 : ea) <= A.lay.size, ST_EINVAL,
                           "gradient plan: operand block out of bounds");
              gp.buf = gp.buf && buffer_reach_ok(GEMM_NN, pb.mi, pb.mj, x.K, x.lda, x.ldb, 8, 8);
            }
            gp.srcs.push_back(x);
          }
        }
        DMRG_REQUIRE(env.chan_off(ch) + ec.nnz <= env.size, ST_EINVAL, "gradient plan: channel out of bounds");
        gp.rows.push_back({env.chan_off(ch), kind_of[cls], 0});
        // flops of this row's products
        const GradSrc* xs = gp.srcs.data() + J.src0 + (long)kind_of[cls] * J.nblk;
        for (int i = 0; i < J.nblk; ++i)
          if (xs[i].valid) gp.flops += 2.0 * pc.blocks[i].mi * pc.blocks[i].mj * xs[i].K;
      }
      gp.units += (long)nr * J.ntile;
      gp.jobs.push_back(J);
    }
  };
  auto run_rows = [&](bool left, GradPlan& gp, GradWork::Tables& t, double* out) {
    if (gp.units == 0) return;
    DMRG_REQUIRE(gp.units < (1L << 31), ST_EINVAL, "too many gradient products in one batch");
    gp.pack();
    t.tables.reserve(gp.packed.size());
    t.units.reserve((size_t)gp.units * sizeof(GemmUnit));
    t.items.reserve((size_t)gp.units * sizeof(GemmItem));
    hip_check(hipMemcpyAsync(t.tables.p, gp.packed.data(), gp.packed.size(), hipMemcpyHostToDevice, st), "grad tables");
    launch_grad_expand(gp.view(t.tables.as<char>()), left, (left ? envl : envr).buf.as<double>(), A.buf.as<double>(),
                       out, t.units.as<GemmUnit>(), t.items.as<GemmItem>(), st);
    launch_gemm_w32(GEMM_NN, gp.buf, t.units.as<GemmUnit>(), (int)gp.units, t.items.as<GemmItem>(), st);
  };
  auto flush = [&]() {
    if (batch.empty()) return;
    // G = P Q^T, K cut into split-K items; the phase's device tables outlive the site
    Phase& pg = grad_.ph;
    pg.mode = GEMM_NT;
    pg.stream = true;
    pg.items.clear();
    pg.units.clear();
    pg.flops = 0;
    pg.uploaded[0] = false;
    for (const Job& jb : batch) {
      const PairClass& pc = classes[jb.c];
      const int ib = (int)pg.items.size();
      for (long k0 = 0; k0 < pc.K; k0 += kGSplit) {
        int kk = (int)std::min<long>(kGSplit, pc.K - k0);
        pg.items.push_back({B_T, jb.poff + k0, B_OUT, jb.qoff + k0, (int)pc.K, (int)pc.K, kk, 1.0});
      }
      pg.units.push_back({B_XMIX, jb.goff, jb.nq, jb.np, jb.nq, 0, 0, ib, (int)pg.items.size(), 0});
      pg.flops += 2.0 * jb.np * jb.nq * (double)pc.K;
    }
    grad_.P.reserve(std::max<long>(bp, 1) * 8);
    grad_.Q.reserve(std::max<long>(bq, 1) * 8);
    grad_.G.reserve(std::max<long>(bg, 1) * 8);
    GradPlan pp, pq;
    void* bases[B_NBUF] = {};
    bases[B_T] = grad_.P.p;
    bases[B_OUT] = grad_.Q.p;
    bases[B_XMIX] = grad_.G.p;
    size_t esz[B_NBUF] = {8, 8, 8, 8, 8, 8, 8, 8, 8};
    long sizes[B_NBUF] = {};
    sizes[B_T] = bp;
    sizes[B_OUT] = bq;
    sizes[B_XMIX] = bg;
    try {
      make_rows(true, pp);
      run_rows(true, pp, grad_.tab[0], grad_.P.as<double>());
      make_rows(false, pq);
      run_rows(false, pq, grad_.tab[1], grad_.Q.as<double>());
      run_phase(pg, PREC_F64, bases, esz, sizes);
    } catch (...) {
      (void)hipStreamSynchronize(st);  // an upload may still read the packed tables
      throw;
    }
    Ghost.resize((size_t)bg);
    hip_check(hipMemcpyAsync(Ghost.data(), grad_.G.p, Ghost.size() * 8, hipMemcpyDeviceToHost, st), "grad G");
    hip_check(hipStreamSynchronize(st), "grad site");  // the packed tables and staging die here
    for (const Job& jb : batch) {
      const int nQ = (int)classes[jb.c].qrow.size();
      for (int r = 0; r < jb.np; ++r)
        std::copy(Ghost.begin() + jb.goff + (size_t)r * jb.nq, Ghost.begin() + jb.goff + (size_t)(r + 1) * jb.nq,
                  Gc[jb.c].begin() + (size_t)(jb.p0 + r) * nQ + jb.q0);
    }
    st_.grad_flops += pp.flops + pq.flops + pg.flops;
    batch.clear();
    bp = bq = bg = 0;
  };
  // all products: classes batched up to `together` doubles of P or Q rows, the rows
  // of a class that alone exceeds `alone` taken in chunks
  auto run_all = [&](long together, long alone) {
    batch.clear();
    bp = bq = bg = 0;
    for (size_t c = 0; c < classes.size(); ++c) {
      const PairClass& pc = classes[c];
      if (pc.prow.empty() || pc.K == 0) continue;
      const int nP = (int)pc.prow.size(), nQ = (int)pc.qrow.size();
      Gc[c].assign((size_t)nP * nQ, 0.0);
      const int cP = (int)std::max<long>(1, std::min<long>(nP, alone / pc.K));
      const int cQ = (int)std::max<long>(1, std::min<long>(nQ, alone / pc.K));
      if (cP == nP && cQ == nQ) {
        const long np = (long)nP * pc.K, nq = (long)nQ * pc.K;
        if (bp + np > together || bq + nq > together) flush();
        batch.push_back({c, 0, nP, 0, nQ, bp, bq, bg, true});
        bp += np;
        bq += nq;
        bg += (long)nP * nQ;
        continue;
      }
      flush();
      for (int p0 = 0; p0 < nP; p0 += cP)
        for (int q0 = 0; q0 < nQ; q0 += cQ) {
          const int np = std::min(cP, nP - p0), nq = std::min(cQ, nQ - q0);
          batch.push_back({c, p0, np, q0, nq, 0, 0, 0, q0 == 0});
          bp = (long)np * pc.K;
          bq = (long)nq * pc.K;
          bg = (long)np * nq;
          flush();
        }
    }
    flush();
  };
  // Where the buffers do not fit (a workspace, a full card), class by class, as
  // little as the gradient ever took, and then half as many rows at a time down to one.
  long largest = 0, deepest = 0;  // of one class: P or Q rows, one row
  for (const PairClass& pc : classes) {
    largest = std::max(largest, pc.K * (long)std::max(pc.prow.size(), pc.qrow.size()));
    deepest = std::max(deepest, pc.K);
  }
  long together = kBatchElems, alone = kChunkElems;
  for (;;) {
    const double flops0 = st_.grad_flops;
    try {
      run_all(together, alone);
      break;
    } catch (const Error& e) {
      if (e.code != ST_ENOMEM || (together == 0 && alone <= deepest)) throw;
      hip_check(hipStreamSynchronize(st), "grad site");
      st_.grad_flops = flops0;
      grad_.release();
      if (together > 0) together = 0;
      else alone = std::max(deepest, std::min(alone, largest) / 2);
    }
  }
  for (size_t e = 0; e < W.size(); ++e)
    for (const Use& u : uses[e]) g[e] += u.w * Gc[u.cls][(size_t)u.pr * (int)classes[u.cls].qrow.size() + u.qr];
  for (const Use& u : norm_uses) *norm += Gc[u.cls][(size_t)u.pr * (int)classes[u.cls].qrow.size() + u.qr];
}

// Per root r with weight w_r != 0: E_r = <Psi_r|H|Psi_r>/<Psi_r|Psi_r> + e_core and
// sum_r w_r dE_r/dh, dE_r/dB (entries of h and B treated as independent).
void Solver::grad(const std::vector<double>& w, std::vector<double>& dh, std::vector<double>& dB,
                  std::vector<double>& energies) {
  const MPO& mpo = prob_->mpo;
  const int n = prob_->n, nq = prob_->nq;
  const bool have_roots = center_site_ >= 0 && (int)centers_.size() == opt_.n_states;
  const int nr = have_roots ? opt_.n_states : 1;
  DMRG_REQUIRE(!w.empty() && (int)w.size() <= opt_.n_states, ST_EINVAL, "one weight per state");
  for (size_t r = (size_t)nr; r < w.size(); ++r)
    DMRG_REQUIRE(w[r] == 0.0, ST_ESTATE, "excited-state gradients need the centre tensors of a sweep");
  for (double x : w) DMRG_REQUIRE(std::isfinite(x), ST_EINVAL, "state weights must be finite");
  dh.assign((size_t)n * n, 0.0);
  dB.assign((size_t)nq * n * n, 0.0);
  energies.assign(w.size(), 0.0);
  std::vector<double> dg;  // d E / d(pq|rs), entries independent
  if (nq > 0) dg.assign((size_t)n * n * n * n, 0.0);
  auto t0 = std::chrono::steady_clock::now();
  GradWork::Use use(grad_);

  const int c = center_site_;
  auto invalidate_around = [&](int site) {
    for (int cut = site + 1; cut <= L_; ++cut) left_[cut].valid = false;
    for (int cut = 0; cut <= site; ++cut) right_[cut].valid = false;
    plan_k_ = -1;
  };
  for (int r = 0; r < nr && r < (int)w.size(); ++r) {  // every root's energy is reported
    if (have_roots && r > 0) {
      launch_copy(mps_[c].buf.as<double>(), centers_[r].as<double>(), center_lay_.size, st);
      invalidate_around(c);
    }
    // g per site, normalised by <Psi|Psi> (the identity path through site 0)
    std::vector<std::vector<double>> gs(L_);
    double norm = 0.0;
    for (int k = 0; k < L_; ++k) grad_site(k, gs[k], k == 0 ? &norm : nullptr);
    DMRG_REQUIRE(norm > 0.0 && std::isfinite(norm), ST_ESTATE, "MPS has zero norm");
    double e0 = 0.0;
    for (size_t e = 0; e < mpo.W[0].size(); ++e) e0 += mpo.W[0][e].c * gs[0][e];
    energies[r] = e0 / norm + prob_->e_core;
    const double wr = w[r] / norm;
    if (wr != 0.0)
      for (int k = 0; k < L_; ++k)
        for (const Prov& p : mpo.prov[k]) {
          double v = wr * p.f * gs[k][p.entry];
          if (p.kind == PK_H) dh[(size_t)p.i[0] * n + p.i[1]] += v;
          else if (p.kind == PK_G) dg[(((size_t)p.i[0] * n + p.i[1]) * n + p.i[2]) * n + p.i[3]] += v;
          else dB[((size_t)p.i[0] * n + p.i[1]) * n + p.i[2]] += v;
        }
    if (have_roots && r > 0) {
      launch_copy(mps_[c].buf.as<double>(), centers_[0].as<double>(), center_lay_.size, st);
      invalidate_around(c);
    }
  }
  // (pq|rs) = sum_Q B^Q_pq B^Q_rs:  dE/dB^Q_ij += sum_rs (dg_ijrs + dg_rsij) B^Q_rs
  const size_t n2 = (size_t)n * n;
  std::vector<double> sym(dg.size()), acc(n2);
  for (size_t ij = 0; ij < n2 && nq > 0; ++ij)
    for (size_t rs = 0; rs < n2; ++rs) sym[rs * n2 + ij] = dg[ij * n2 + rs] + dg[rs * n2 + ij];
  for (int q = 0; q < nq; ++q) {
    const double* Bq = prob_->B.data() + (size_t)q * n2;
    double* out = dB.data() + (size_t)q * n2;
    std::fill(acc.begin(), acc.end(), 0.0);
    for (size_t rs = 0; rs < n2; ++rs)
      for (size_t ij = 0; ij < n2; ++ij) acc[ij] += sym[rs * n2 + ij] * Bq[rs];
    for (size_t ij = 0; ij < n2; ++ij) out[ij] += acc[ij];
  }
  // small buffers stay for the next call; a workspace gets everything back
  if (current_arena() || grad_.bytes() > kKeepBytes) grad_.release();
  st_.grad_ms += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
}

// Two-orbital density matrices of the stored MPS (root 0), every pair i < j, in
// the determinant convention of the CI route (local creators moved to the front
// in the order i alpha, j alpha, i beta, j beta): each element is the
// derivative of <Psi|O|Psi> by one closing entry of the pair MPO (the same
// per-site contractions as the integral gradient), over <Psi|Psi>.  The MPO
// gives them with the site creators in chain order (i alpha, i beta, j alpha,
// j beta); reordering to the determinant convention flips the sign of a local
// state holding beta on i and alpha on j.
std::vector<double> Solver::pair_rdm_mps() {
  materialize();
  Problem p2;
  p2.n = L_;
  p2.n_alpha = prob_->n_alpha;
  p2.n_beta = prob_->n_beta;
  std::vector<PairClosing> closings;
  p2.mpo = build_pair_mpo(L_, closings);
  Options o;
  o.M = 1;
  Solver s2(&p2, o, st);
  s2.adopt_mps(*this);
  s2.centers_.clear();  // the MPS as stored
  std::vector<std::vector<double>> gs(L_);
  double norm = 0.0;
  for (int k = 0; k < L_; ++k) s2.grad_site(k, gs[k], k == 0 ? &norm : nullptr);
  DMRG_REQUIRE(norm > 0.0 && std::isfinite(norm), ST_ESTATE, "MPS has zero norm");
  const int np = L_ * (L_ - 1) / 2;
  std::vector<double> rho((size_t)np * 256, 0.0);
  auto pair_index = [&](int i, int j) { return i * L_ - i * (i + 1) / 2 + (j - i - 1); };
  auto tau = [](int ti, int tj) { return ((ti & 2) && (tj & 1)) ? -1.0 : 1.0; };
  for (const PairClosing& c : closings) {
    const int Lb = c.t + 4 * c.tj, Lk = c.s + 4 * c.sj;
    rho[(size_t)pair_index(c.i, c.j) * 256 + Lb * 16 + Lk] =
        tau(c.t, c.tj) * tau(c.s, c.sj) * gs[c.j][c.entry] / norm;
  }
  return rho;
}

}  // namespace dmrg
