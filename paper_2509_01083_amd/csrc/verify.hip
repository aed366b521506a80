// Batched speculative verification with ragged per-sequence speculation
// lengths on gfx950 (speculative sampling, Sec. 2.1; ragged layout, bonus and
// pad, Sec. 3.2; per-token KLD of the SL adapter, Sec. 3.1.2).
//
// Kernels, in launch order on the caller's stream:
//   setup_kernel, stats_kernel   (stats.hip) layout check, work list, and the
//                      row statistics of every drafted pair, chunk by chunk
//                      (small batches: no set-up kernel, seq_kernel checks the
//                      layout).
//   seq_kernel         several workgroups per sequence.  Each combines the chunk
//                      partials of the sequence's drafted pairs (fp64) and finds
//                      the acceptance u < p(x)/q(x) (fp64) up to the first
//                      rejection.  One of them writes the outputs (accepted
//                      drafts, KLD, and in the fused step the signal update);
//                      the others stream the draw's row(s), the residual
//                      max(0, p - q) of the rejected pair or the bonus row, and
//                      leave weight totals per unit of 2048 logits.
//   pick_kernel        one workgroup per sequence: the token, by a fixed-order
//                      fp64 prefix over the units to the one holding u' * Z, the
//                      same over its four sub-blocks, and an ordered scan of the
//                      512 logits of the sub-block found.  Fused step: one more
//                      workgroup runs the batch cap and the next lengths, which
//                      need nothing from the draw.
//
// Every reduction runs in a fixed order, so results are bitwise reproducible.
#include <math.h>

#include "common.hpp"
#include "draw_device.hpp"
#include "row_io.hpp"
#include "signal_device.hpp"

namespace dsde {
namespace {

constexpr int kSeqThreads = 256;
constexpr int kSeqWaves = kSeqThreads / 64;
constexpr int kSignalWave = kSeqWaves - 1;  // wavefront of the KLD outputs and the fused signal update

struct StepParams {
  const void *target, *draft;
  int64_t V;
  int32_t B, k_max, nc, nu, pad_id;
  bool lookup;        // no set-up kernel ran: this kernel checks the layout and writes seq_err
  int64_t N;
  int32_t first_seq;  // first sequence of this pass (the cells and jobs are indexed from it)
  const int32_t *sl, *cu_sl, *draft_tokens;
  const float *temperature, *u_acc, *u_res;
  int32_t *accepted, *tokens;
  float *kld;
  uint32_t *seq_err;
  double *row_lse;
  float *entropy;  // draft entropy per drafted position (nats), may be null
  const PairChunk *part;
  const Gathered *gathered;
  const ChunkArg *chunk_arg;  // greedy pairs: the target row's maximum and argmax per chunk
  DrawJob *jobs;
  float *sub;
  UnitRef *ref;
};

// ---------------------------------------------------------------------------
// acceptance, outputs and draw weights
// ---------------------------------------------------------------------------

// Workgroup (x, y) works on one sequence of the pass; y = 0 writes the outputs,
// y = 1 .. gridDim.y - 1 take a share of the draw's units each (MERGED, for many
// sequences: y = 0 too).  All of them
// repeat the acceptance: it takes about 3 us of latency and few instructions,
// where handing its result to other workgroups would take a kernel boundary.
// A row dealt to one workgroup per sequence is bound by that CU's VALU (two
// exponentials per logit pair), 20 us for two bf16 rows of 128,256 logits, and
// leaves the other CUs idle in small batches.  Measured against the kernel that
// streamed and drew in one workgroup per sequence: 21.7 -> 6.6 us for one
// sequence (V = 128,256 bf16), 65.4 -> 14.6 us for 64 in fp32,
// 29.8 -> 25.8 us for 256 in bf16 (18 us of bytes).
template <int DT, int ROW, bool FUSED, bool MERGED>
__global__ __launch_bounds__(kSeqThreads) void seq_kernel(const StepParams P, const SignalArgs S) {
  __shared__ float st_mt[DSDE_MAX_K + 1], st_md[DSDE_MAX_K + 1];
  __shared__ double st_sp[DSDE_MAX_K + 1], st_sq[DSDE_MAX_K + 1], st_a[DSDE_MAX_K + 1], st_h[DSDE_MAX_K + 1];
  __shared__ int st_bad[DSDE_MAX_K + 1], st_arg[DSDE_MAX_K + 1];
  __shared__ uint32_t s_err_in, s_err;  // error bits before and after the row checks
  __shared__ DrawJob s_job;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);  // uniform: unit indices and addresses stay scalar
  // last sequence first: its rows are what the statistics pass read last.  Worth
  // 0.5 % of a 256-sequence step; second reads of rows come at the speed of the
  // first, so it is not the last-level cache serving them that gives it.
  const int32_t lb = int32_t(gridDim.x) - 1 - int32_t(blockIdx.x), b = P.first_seq + lb;
  const bool outputs = blockIdx.y == 0;
  const int32_t width = P.k_max + 1;
  int32_t *tok = P.tokens + int64_t(b) * width;
  // first round trip: everything whose address depends on the sequence index
  // alone - this sequence's chunk partials and gathered logits (stored by slot
  // b * k_max + j; positions past SL_b are fetched and ignored), and the
  // per-sequence inputs
  const int G = P.nc <= 16 ? 16 : P.nc <= 32 ? 32 : 64;
  const int32_t j0 = wave * (64 / G) + lane / G, g0 = lane % G;
  const int64_t slot0 = int64_t(b) * P.k_max;
  PairChunk q0{};
  if (j0 < P.k_max && g0 < P.nc) q0 = P.part[(slot0 + j0) * P.nc + g0];
  ChunkArg arg0{0.f, 0};  // greedy pairs only; fetched regardless, it costs no extra round trip
  if (j0 < P.k_max && g0 < P.nc) arg0 = P.chunk_arg[(slot0 + j0) * P.nc + g0];
  Gathered gz{0.f, 0.f};
  if (wave == 0 && lane < P.k_max) gz = P.gathered[slot0 + lane];
  const int32_t s = P.sl[b], first = P.cu_sl[b];
  const float T = P.temperature[b], ur = P.u_res[b];
  RingPrefetch<1> rp{};
  if constexpr (FUSED)
    if (outputs && wave == kSignalWave)
      rp = wave_ring_prefetch<1>(S.hist + int64_t(b) * S.W, S.head + b, S.count + b, S.W);
  // without a set-up kernel the outputs workgroup checks the whole layout, here
  // beside the first round trip; the streaming ones look only at what keeps
  // their own reads in bounds (their cells go unused when the layout is invalid)
  const int fault = P.lookup && outputs ? layout_fault(P.B, P.N, P.k_max, P.sl, P.cu_sl) : 0;
  // one wait for the whole first round trip: every load above is issued
  // before any of the pins below asks for its value
  asm volatile("" ::: "memory");
  pin(q0.mt);
  pin(q0.md);
  pin(q0.sp);
  pin(q0.sq);
  pin(q0.a);
  pin(gz.zt);
  pin(gz.zd);
  pin(arg0.zmax);
  pin(arg0.idx);
  const bool own_bad = P.lookup ? s < 0 || s > P.k_max || first < 0 || int64_t(first) + s > P.N
                                : (P.seq_err[b] & DSDE_ERR_LAYOUT) != 0;
  if (!outputs && own_bad) return;
  if (outputs && (P.lookup ? __syncthreads_or(fault) != 0 : own_bad)) {
    if (t < width) tok[t] = P.pad_id;
    if (t == 0) {
      if (P.lookup) P.seq_err[b] = DSDE_ERR_LAYOUT;
      P.accepted[b] = 0;
      DrawJob j{};
      j.kind = -1;
      P.jobs[lb] = j;
      if constexpr (FUSED) S.mu_last[b] = S.var_short[b] = S.var_long[b] = S.wvir[b] = S.sf[b] = NAN;
    }
    return;
  }
  // T_b = 0: greedy verification (statistics at T = 1, uniforms unused)
  const bool greedy = T == 0.0f;
  const ChunkArg *cargs = greedy ? P.chunk_arg : nullptr;
  // per-position inputs of wavefront 0 (lane j = drafted position j)
  int32_t x = 0;
  float u = 0.f;
  if (wave == 0 && lane < s) {
    x = P.draft_tokens[first + lane];
    u = P.u_acc[first + lane];
  }

  // ---- acceptance
  // row statistics of every drafted pair (read even for a flagged sequence:
  // the layout is valid, so every access stays in bounds)
  if (s > 0) {
    if (G == 16)
      combine_pairs<16, kSeqWaves>(P.part, slot0, s, P.nc, q0, cargs, arg0, st_mt, st_md, st_sp, st_sq, st_a,
                                    st_h, st_bad, st_arg);
    else if (G == 32)
      combine_pairs<32, kSeqWaves>(P.part, slot0, s, P.nc, q0, cargs, arg0, st_mt, st_md, st_sp, st_sq, st_a,
                                    st_h, st_bad, st_arg);
    else
      combine_pairs<64, kSeqWaves>(P.part, slot0, s, P.nc, q0, cargs, arg0, st_mt, st_md, st_sp, st_sq, st_a,
                                    st_h, st_bad, st_arg);
  }
  __syncthreads();
  // the outputs workgroup's last wavefront forms the KLD of every drafted
  // position (lane j: position j), its draft entropy and row log-normalisers
  // beside wavefront 0's acceptance, and writes them behind the barrier, where
  // the error bits are known
  double my_kl = 0.0, my_h = 0.0, lse_t = 0.0, lse_d = 0.0;
  if (outputs && wave == kSignalWave && lane < s) {
    const double sp = st_sp[lane], sq = st_sq[lane];
    const double l2sp = log2_rowsum(sp), l2sq = log2_rowsum(sq);
    // KL in log2 units: E_p[(z_t c - mt) - (z_d c - md)] - log2 S_p + log2 S_q
    my_kl = (st_a[lane] * rcp_newton(sp) - l2sp + l2sq) * kLn2;
    // draft entropy in log2 units: log2 S_q - E_q[z_d c - md]
    my_h = (l2sq - st_h[lane] * rcp_newton(sq)) * kLn2;
    lse_t = (double(st_mt[lane]) + l2sp) * kLn2;
    lse_d = (double(st_md[lane]) + l2sq) * kLn2;
  }
  if (wave == 0) {
    uint32_t err = 0;
    {  // per-sequence input checks
      uint32_t e = 0;
      if (lane < s) {
        if (x < 0 || int64_t(x) >= P.V) e |= DSDE_ERR_TOKEN;
        if (!greedy && !(u >= 0.0f && u < 1.0f)) e |= DSDE_ERR_UNIFORM;
      }
      if (lane == 0 && !greedy) {
        if (!(T >= kMinTemp && T <= kMaxTemp)) e |= DSDE_ERR_TEMP;
        if (!(ur >= 0.0f && ur < 1.0f)) e |= DSDE_ERR_UNIFORM;
      }
      err |= lanes::wave_or(e);
    }
    const float c = greedy ? kLog2e : kLog2e / T;  // the same values as the set-up's scale
    const bool active = lane < s && !err;
    bool ok = false, bad = false;
    float my_mt = 0.f, my_md = 0.f, my_isp = 0.f, my_isq = 0.f;
    int32_t my_arg = 0;
    if (lane == 0) s_err_in = err;  // the KLD wavefront writes the log-normalisers of unflagged sequences
    if (active) {
      bad = st_bad[lane] != 0;
      const double sp = st_sp[lane], sq = st_sq[lane];
      my_mt = st_mt[lane];
      my_md = st_md[lane];
      my_arg = st_arg[lane];
      my_isp = float(rcp_newton(sp));
      my_isq = float(rcp_newton(sq));
      if (greedy) {
        ok = x == my_arg;  // accept iff the drafted token is the target row's argmax
      } else {
        // u < p(x) / q(x) with p(x) = 2^(z_t(x) c - mt) / S_p and q(x) = 2^(z_d(x) c - md) / S_q,
        // tested as u S_p < 2^D S_q (no logarithm on this path; z c is exact in double)
        const double D = (double(gz.zt) * double(c) - double(my_mt)) - (double(gz.zd) * double(c) - double(my_md));
        ok = double(u) * sp < exp2_taylor(D) * sq;
      }
    }
    if (__ballot(bad)) err |= DSDE_ERR_LOGIT;
    const uint64_t mask = __ballot(ok);
    int32_t a = int32_t(__builtin_ctzll(~mask));
    if (a > s) a = s;
    if (err) a = 0;
    if (lane == 0) s_err = err;
    // the first rejected position's row values, from its lane
    const float a_mt = lanes::readlane(my_mt, a), a_md = lanes::readlane(my_md, a);
    const float a_isp = lanes::readlane(my_isp, a), a_isq = lanes::readlane(my_isq, a);
    const int32_t a_arg = lanes::readlane(my_arg, a);
    DrawJob j{};
    j.kind = -1;
    if (!err && greedy) {
      j.accepted = a;
      j.target_row = first + b + a;
      j.draft_row = -1;
      if (a < s) {  // the argmax of the first rejected row is known already
        j.kind = 2;
        j.token = a_arg;
      } else {      // the argmax of the bonus row
        j.kind = 3;
      }
    } else if (!err) {
      j.accepted = a;
      j.scale = c;
      j.u = ur;
      if (a < s) {
        j.kind = 0;
        j.target_row = first + b + a;
        j.draft_row = first + a;
        j.mt = a_mt;
        j.md = a_md;
        j.inv_sp = a_isp;
        j.inv_sq = a_isq;
      } else {
        j.kind = 1;
        j.target_row = first + b + s;
        j.draft_row = -1;
      }
    }
    if (outputs) {
      if (lane < width) tok[lane] = lane < a ? x : j.kind == 2 && lane == a ? j.token : P.pad_id;
      if (lane == 0) {
        P.accepted[b] = a;
        P.jobs[lb] = j;
        if (P.lookup)
          P.seq_err[b] = err;  // ahead of the barrier below, behind which the signal's bits are OR-ed in
        else if (err)
          atomicOr(&P.seq_err[b], err);
      }
      if constexpr (MERGED)
        if (lane == 0) s_job = j;
    } else if (lane == 0) {
      s_job = j;
    }
  }
  __syncthreads();

  if (MERGED || !outputs) {
    // ---- this workgroup's share of the draw's units
    const DrawJob job = uniform_job(s_job);
    const UnitCells cells{P.sub + int64_t(lb) * P.nu * kSubs, P.ref + int64_t(lb) * P.nu};
    const int32_t gw = (int32_t(blockIdx.y) - !MERGED) * kSeqWaves + wave;
    draw_units<DT, ROW>(job, (const char *)P.target, (const char *)P.draft, P.V, P.nu, gw,
                        (int32_t(gridDim.y) - !MERGED) * kSeqWaves, cells);
    if (!outputs) return;
  }
  if (wave != kSignalWave) return;
  // ---- the KLD outputs, and in the fused step the signal update of Sec. 3.1.2
  // on those KLD values
  const uint32_t e_in = s_err_in, e_all = s_err;
  const float my_kld = e_all ? NAN : my_kl > 0.0 ? float(my_kl) : 0.0f;
  if (lane < s) {
    P.kld[first + lane] = my_kld;
    if (P.entropy) P.entropy[first + lane] = e_all ? NAN : float(my_h);
    if (P.row_lse && !e_in && !st_bad[lane]) {
      P.row_lse[2 * (first + lane)] = lse_t;
      P.row_lse[2 * (first + lane) + 1] = lse_d;
    }
  }
  if constexpr (FUSED) {
    const uint32_t e = wave_signal_update(s, first, nullptr, my_kld, rp, S.hist + int64_t(b) * S.W, S.head + b,
                                          S.count + b, S.W, S.n_short, S.n_long, S.delta, S.eps, S.mu_last + b,
                                          S.var_short + b, S.var_long + b, S.wvir + b, S.sf + b);
    if (e && lane == 0) atomicOr(&P.seq_err[b], e);
  }
}

// ---------------------------------------------------------------------------
// the drawn token
// ---------------------------------------------------------------------------

// One workgroup per sequence of the pass; with `rule` set, workgroup gridDim.x
// - 1 is the SL rule's (the same workgroup size as next_sl_kernel, so the same
// order of its sums).  A sequence's draw needs one wavefront; the others are
// there for a residual without mass, whose fallback to p has to read the
// target row again.
template <int DT, int ROW>
__global__ __launch_bounds__(kCapThreads) void pick_kernel(const StepParams P, const SignalArgs S, bool rule) {
  if (rule && blockIdx.x == gridDim.x - 1) {
    __shared__ double red_s[kCapThreads / 64];
    __shared__ int red_n[kCapThreads / 64];
    block_next_sl(P.B, S.sf, S.wvir, S.sl_max, S.sl_min, S.sl_hi, S.budget, S.sl_hat, S.sl_cap, S.sl_next, P.seq_err,
                  true, red_s, red_n);
    return;
  }
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int32_t lb = blockIdx.x, b = P.first_seq + lb;
  const UnitCells cells{P.sub + int64_t(lb) * P.nu * kSubs, P.ref + int64_t(lb) * P.nu};
  // one round trip: the job and the first 64 units' cells (whatever they hold
  // when the job does not use them)
  UnitCell cell0 = load_cell(cells, lane, P.nu, true);
  const DrawJob job = uniform_job(P.jobs[lb]);
  if (job.kind < 0 || job.kind == 2) return;  // flagged, or a greedy token already emitted
  const int32_t width = P.k_max + 1;
  int32_t *tok = P.tokens + int64_t(b) * width;
  int mode = job.kind == 0 ? 0 : 2;  // 0: residual weights, 1: p of the rejected pair, 2: bonus exponentials
  float row_ref = 0.f;
  double Z = 0.0;  // the row's total weight
  if (job.kind != 0) {
    bool bad;
    row_ref = row_reference(cells, P.nu, cell0, &bad);
    if (wave != 0) return;
    if (job.kind == 1) {
      Z = row_total(cells, P.nu, cell0, mode, row_ref);
      bad |= !(Z > 0.0);
    }
    if (bad) {
      // a NaN or infinite logit in the bonus row, or no weight in it: no token is emitted
      if (lane < width) tok[lane] = P.pad_id;
      if (lane == 0) {
        P.accepted[b] = 0;
        atomicOr(&P.seq_err[b], DSDE_ERR_LOGIT);
      }
      return;
    }
    if (job.kind == 3) {
      const int32_t token = row_argmax(cells, P.nu, cell0, row_ref);
      if (lane == 0) tok[job.accepted] = token;
      return;
    }
  }
  const size_t esz = DT == DSDE_BF16 ? 2 : 4;
  const char *trow = (const char *)P.target + size_t(job.target_row) * size_t(P.V) * esz;
  const char *drow =
      job.kind == 0 ? (const char *)P.draft + size_t(job.draft_row) * size_t(P.V) * esz : nullptr;
  if (mode == 0) Z = row_total(cells, P.nu, cell0, mode, row_ref);
  if (mode == 0 && !(Z > 0.0)) {  // no residual mass (the same in every wavefront): p of the same target row
    mode = 1;
    __syncthreads();  // every wavefront has read the residual's cells, which p's now replace
    for (int32_t u = wave; u < P.nu; u += kCapThreads / 64) target_p_unit<DT, ROW>(trow, P.V, u, job, cells);
    __syncthreads();
    cell0 = load_cell(cells, lane, P.nu, false);
    Z = row_total(cells, P.nu, cell0, mode, row_ref);
  }
  if (wave != 0) return;
  const int32_t token =
      draw_in_row<DT, ROW>(cells, P.nu, cell0, row_ref, double(job.u) * Z, trow, drow, P.V, mode, job);
  if (lane == 0) tok[job.accepted] = token;
}

}  // namespace

// Streaming workgroups per sequence.  Up to kStreamWorkgroups sequences: about
// that many workgroups in all, but no wavefront without a unit.  Five of them fit
// a CU by registers (aligned rows), 1,280 the chip, where the outputs workgroups
// need places too: 1,280 and 2,048 streaming ones were slower (256 sequences at
// V = 128,256: 127.5 and 128.9 us a step against 125.8; 512 long drafts: 490 and
// 487 against 483; 1,024 of 2-3 drafts: 298 and 299 against 290).
// More sequences: the outputs workgroups stream as well (MERGED), since a round of
// workgroups that only decide, ahead of those that stream, leaves memory idle, and
// each workgroup takes about 32 units, so that the acceptance it repeats stays small
// and the last round of workgroups short.  V = 128,256, 1-2 drafts: 1,536
// sequences 316 -> 302 us, 2,048 410 -> 400, 4,096 830 -> 790; V = 32,000, 1-4
// drafts: 4,096 323 -> 314 us; 65,536 at V = 512: 1,277 -> 1,086 us.
constexpr int32_t kStreamWorkgroups = 1024;
static int32_t stream_parts(int32_t seqs, int32_t nu) {
  if (seqs > kStreamWorkgroups) return nu < 48 ? 1 : (nu + 16) / 32;
  const int32_t most = (nu + kSeqWaves - 1) / kSeqWaves;
  const int32_t want = (kStreamWorkgroups + seqs - 1) / seqs;
  return want < most ? want : most;
}

template <int DT, int ROW>
static void launch_draw(const VerifyArgs &a, StepParams P, const SignalArgs &S) {
  const int32_t per_pass = draw_seqs_per_pass(a.B, a.V);
  for (int32_t b0 = 0; b0 < a.B; b0 += per_pass) {
    const int32_t seqs = a.B - b0 < per_pass ? a.B - b0 : per_pass;
    const bool last = b0 + seqs == a.B;
    P.first_seq = b0;
    const bool merged = seqs > kStreamWorkgroups;
    const dim3 grid(unsigned(seqs), unsigned(stream_parts(seqs, P.nu) + !merged));
    auto run = [&](auto kernel) { kernel<<<grid, dim3(kSeqThreads), 0, a.stream>>>(P, S); };
    if (a.signal)
      merged ? run(seq_kernel<DT, ROW, true, true>) : run(seq_kernel<DT, ROW, true, false>);
    else
      merged ? run(seq_kernel<DT, ROW, false, true>) : run(seq_kernel<DT, ROW, false, false>);
    // the SL rule needs every sequence's signal: behind the last pass
    const bool rule = a.signal && last;
    pick_kernel<DT, ROW><<<dim3(unsigned(seqs + rule)), dim3(kCapThreads), 0, a.stream>>>(P, S, rule);
  }
}

int launch_verify(const VerifyArgs &a) {
  const WorkspaceLayout L = workspace_layout(a.B, a.N, a.V, a.k_max);
  char *ws = (char *)a.workspace;
  WorkItem *work = (WorkItem *)(ws + L.work);
  PairChunk *part = (PairChunk *)(ws + L.pair_chunk);
  Gathered *gath = (Gathered *)(ws + L.gathered);
  (void)hipGetLastError();
  ChunkArg *cargs = (ChunkArg *)(ws + L.chunk_arg);
  const bool lookup = stats_lookup(a);
  launch_stats_pass(a, lookup, work, part, gath, cargs, a.draft_entropy != nullptr);
  StepParams P;
  P.target = a.target;
  P.draft = a.draft;
  P.V = a.V;
  P.B = a.B;
  P.k_max = a.k_max;
  P.nc = int32_t(num_chunks(a.V));
  P.nu = int32_t(num_units(a.V));
  P.pad_id = a.pad_id;
  P.lookup = lookup;
  P.N = a.N;
  P.first_seq = 0;
  P.sl = a.sl;
  P.cu_sl = a.cu_sl;
  P.draft_tokens = a.draft_tokens;
  P.temperature = a.temperature;
  P.u_acc = a.u_acc;
  P.u_res = a.u_res;
  P.accepted = a.accepted;
  P.tokens = a.tokens;
  P.kld = a.kld;
  P.seq_err = a.seq_err;
  P.row_lse = a.row_lse;
  P.entropy = a.draft_entropy;
  P.part = part;
  P.gathered = gath;
  P.chunk_arg = cargs;
  P.jobs = (DrawJob *)(ws + L.jobs);
  P.sub = (float *)(ws + L.sub);
  P.ref = (UnitRef *)(ws + L.ref);
  const SignalArgs S = a.signal ? *a.signal : SignalArgs{};
  by_rows(a.dtype, rows_form(a.target, a.draft, a.dtype, a.V, a.N),
          [&](auto dt, auto row) { launch_draw<decltype(dt)::value, decltype(row)::value>(a, P, S); });
  return hipGetLastError() == hipSuccess ? DSDE_OK : DSDE_DEVICE_ERROR;
}

}  // namespace dsde
