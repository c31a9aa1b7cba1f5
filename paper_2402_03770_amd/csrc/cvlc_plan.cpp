// Host-side code-length planner of libcvlc: plan construction for the three
// ways a caller can fix the plan (given fractions, given code lengths plus a
// budget, or Algorithm 1), plan validation and gamma of Eq. (5).
//
// Accounting follows Eq. (3): every coded group gets the same bit share b (the
// paper's equal packet size, scaled up to a run of packets), pays H = 128 bits
// for its header and (s + y_r) bits per update; the stream adds one 256-bit
// global header.
#include <sched.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <limits>
#include <thread>
#include <vector>

#include "cvlc_common.h"

namespace {

using cvlc::kGlobalHeaderBits;
using cvlc::kSegHeaderBits;

struct PowerLaw {  // Definition 1 with beta = 2*alpha + 1: energy of ranks (lo, hi] over the total
  double d, beta, denom;
  bool log_limit;
  PowerLaw(double d_, double alpha) : d(d_), beta(2.0 * alpha + 1.0) {
    log_limit = std::fabs(beta) < 1e-9;
    denom = log_limit ? std::log(d) : std::pow(d, beta) - 1.0;
  }
  // what share() takes the difference of; a caller that keeps one end of a range keeps its value
  double term(double z) const {
    z = z < 1.0 ? 1.0 : z;  // Z_0 = 0 is read as rank 1 (the power law starts at l = 1)
    return log_limit ? std::log(z) : std::pow(z, beta);
  }
  double share(double hi, double lo) const { return (term(hi) - term(lo)) / denom; }
};

// PQ: Q(P, y) = P / (2^y - 1)^2 (Appendix, case study).
double pq_error(double P, double y) {
  if (!(y > 0.0)) return std::numeric_limits<double>::infinity();
  const double levels = std::exp2(y) - 1.0;
  return P / (levels * levels);
}

// QSGD: Q(P, y) = min(P / s^2, sqrt(P) / s) (Appendix, case study), s = 2^(y-1) - 1 the
// levels above zero that y bits hold beside the sign.
double qsgd_error(double P, double y) {
  if (!(y > 1.0)) return std::numeric_limits<double>::infinity();
  const double levels = std::exp2(y - 1.0) - 1.0;
  const double a = P / (levels * levels), b = std::sqrt(P) / levels;
  return a < b ? a : b;
}

struct ErrorModel {  // the bracket (Q/B^2 + 1/B_c^2) of Eq. (5)/(6), 1/B + 1/B_c = 1
  double inv_b2, inv_bc2;
  uint32_t quant;
  explicit ErrorModel(double B, uint32_t quant_ = CVLC_QUANT_PQ) : inv_b2(1.0 / (B * B)), quant(quant_) {
    const double inv_bc = 1.0 - 1.0 / B;
    inv_bc2 = inv_bc * inv_bc;
  }
  double weight(double P, double y) const {
    return (quant == CVLC_QUANT_QSGD ? qsgd_error(P, y) : pq_error(P, y)) * inv_b2 + inv_bc2;
  }
};

double gamma_integer(uint32_t d, uint32_t R, const uint32_t* P, const uint32_t* y, double alpha, double B,
                     uint32_t quant = CVLC_QUANT_PQ) {
  const PowerLaw law((double)d, alpha);
  const ErrorModel err(B, quant);
  double k = 0.0;
  for (uint32_t r = 0; r < R; ++r) k += (double)P[r];
  // ranks k+1..d are sparsified away; with k = d there are none
  double g = k >= (double)d ? 0.0 : law.share((double)d, k + 1.0);
  double z_prev = 0.0;
  for (uint32_t r = 0; r < R; ++r) {
    const double z = z_prev + (double)P[r];
    if (P[r] > 0) g += err.weight((double)P[r], (double)y[r]) * law.share(z, z_prev);
    z_prev = z;
  }
  return g;
}

int64_t group_share_bits(uint64_t budget_bits, uint32_t R) {
  if (R == 0 || budget_bits < kGlobalHeaderBits) return -1;
  return (int64_t)(32u * ((budget_bits - kGlobalHeaderBits) / (32u * (uint64_t)R)));
}

void plan_init(cvlc_plan_t* p, uint32_t d, uint32_t R, float B) {
  std::memset(p, 0, sizeof(*p));
  p->d = d;
  p->n_coded = R;
  p->s = cvlc::position_bits(d);
  p->B = B;
  p->quant = 0;
}

int plan_from_fractions(uint32_t d, uint32_t R, const uint32_t* y, const double* frac, float B, cvlc_plan_t* out) {
  plan_init(out, d, R, B);
  double cum = 0.0;
  uint64_t z_prev = 0;
  for (uint32_t r = 0; r < R; ++r) {
    if (!(frac[r] >= 0.0)) return CVLC_ERR_ARG;
    cum += frac[r];
    double zf = std::floor((double)d * cum);
    if (zf > (double)d) zf = (double)d;
    uint64_t z = (uint64_t)zf;
    if (z < z_prev) z = z_prev;
    out->code_len[r] = y[r];
    out->count[r] = (uint32_t)(z - z_prev);
    z_prev = z;
  }
  out->total_bits = cvlc_plan_total_bits(out);
  return cvlc_plan_validate(out);
}

int plan_from_budget(uint32_t d, uint64_t budget, uint32_t R, const uint32_t* y, float B, cvlc_plan_t* out) {
  if (R < 1) return CVLC_ERR_ARG;
  plan_init(out, d, R, B);
  const int64_t b = group_share_bits(budget, R);
  if (b < (int64_t)kSegHeaderBits) return CVLC_ERR_BUDGET;
  uint64_t room = d, k = 0;
  for (uint32_t r = 0; r < R; ++r) {
    if (!cvlc::code_len_supported(y[r])) return CVLC_ERR_PLAN;
    uint64_t P = (uint64_t)(b - kSegHeaderBits) / (out->s + y[r]);
    if (P > room) P = room;
    out->code_len[r] = y[r];
    out->count[r] = (uint32_t)P;
    room -= P;
    k += P;
  }
  if (k < R && d >= R) return CVLC_ERR_BUDGET;
  out->total_bits = cvlc_plan_total_bits(out);
  if (out->total_bits > budget) return CVLC_ERR_BUDGET;
  return cvlc_plan_validate(out);
}

// One instance of problem P2 for a fixed budget share: Algorithm 1.
class Algorithm1 {
 public:
  Algorithm1(uint32_t d, uint32_t R, uint32_t s, double usable_bits, double alpha, double B, uint32_t quant)
      : d_(d), R_(R), s_(s), u_(usable_bits), law_((double)d, alpha), err_(B, quant), alpha_(alpha), B_(B),
        quant_(quant), y_min_(quant == CVLC_QUANT_QSGD ? 2.0 : 1.0),
        by_slope_(quant == CVLC_QUANT_PQ && err_.inv_bc2 == 0.0 && alpha >= -4.0 && alpha < 0.0 &&
                  (law_.log_limit || std::fabs(law_.beta) > 1e-3)) {}

  // f(X, P_{r-1}, P_r) of Eq. (6) as a function of P_r: the pair's outer ends stay, and so do their power-law terms.
  struct Pair {
    double X, z_r2, term_r, term_r2;
  };
  Pair pair(double X, double z_r2) const { return Pair{X, z_r2, law_.term(z_r2 + X), law_.term(z_r2)}; }
  double pair_cost(double Pr, const Pair& pr) const {
    const double Pr1 = pr.X - Pr;
    const double term_r1 = law_.term(pr.z_r2 + Pr1);
    const double a = err_.weight(Pr, u_ / Pr - (double)s_) * ((pr.term_r - term_r1) / law_.denom);
    const double b = err_.weight(Pr1, u_ / Pr1 - (double)s_) * ((term_r1 - pr.term_r2) / law_.denom);
    return a + b;
  }

  // Derivative of pair_cost (PQ) by Pr.  With L = 2^y - 1 and y = u/P - s the weight P/L^2/B^2 grows as
  // (1 + 2 ln2 (1 + 1/L) u/P) / L^2 / B^2; the power-law term's own derivative is beta times the term over its rank.
  double pair_slope(double Pr, const Pair& pr) const {
    const double Pr1 = pr.X - Pr, Z = pr.z_r2 + Pr1;
    const double term_r1 = law_.term(Z);
    const double fall = Z < 1.0 ? 0.0 : (law_.log_limit ? 1.0 / Z : law_.beta * term_r1 / Z);  // term_r1 falls by this as Pr grows
    auto weight = [&](double P, double* grows) {
      const double bits = u_ / P, y = bits - (double)s_;
      const double levels = std::exp2(y) - 1.0, unit = err_.inv_b2 / (levels * levels);
      *grows = unit * (1.0 + 1.3862943611198906 * (1.0 + 1.0 / levels) * bits);
      return P * unit + err_.inv_bc2;
    };
    double grows, grows1;
    const double w = weight(Pr, &grows), w1 = weight(Pr1, &grows1);
    return (grows * (pr.term_r - term_r1) + w * fall - grows1 * (term_r1 - pr.term_r2) - w1 * fall) / law_.denom;
  }

  // Zero of pair_slope in [lo, hi], or the end that the cost falls towards, from x on: secant steps inside what is known to hold the
  // zero, halving it where they do not help.  NaN if the slope is not a number somewhere.
  double flat_point(double lo, double hi, double x, const Pair& pr) const {
    double a = lo, b = hi, x_before = 0.0, g_before = 0.0, width = 2.0 * (hi - lo);
    bool a_known = false, b_known = false, one = false;  // whether the slope has been seen below 0 at a, above 0 at b, and anywhere
    x = std::min(std::max(x, lo), hi);
    const double close = 1e-11 * hi;
    for (int it = 0; it < 200; ++it) {
      const double g = pair_slope(x, pr);
      if (!(std::fabs(g) <= std::numeric_limits<double>::max())) return std::numeric_limits<double>::quiet_NaN();
      if (g == 0.0) return x;
      if (g < 0.0) {
        if (x == hi) return hi;
        a = x;
        a_known = true;
      } else {
        if (x == lo) return lo;
        b = x;
        b_known = true;
      }
      double next = one ? x - g * (x - x_before) / (g - g_before) : x - (g < 0.0 ? -1.0 : 1.0) * 1e-3 * (hi - lo);
      const bool halve = it % 4 == 3 && a_known && b_known && b - a > 0.5 * width;
      if (it % 4 == 3) width = b - a;
      x_before = x;
      g_before = g;
      one = true;
      if (!(next > a)) next = a_known ? a + 0.5 * (b - a) : lo;
      else if (!(next < b)) next = b_known ? a + 0.5 * (b - a) : hi;
      else if (halve) next = a + 0.5 * (b - a);
      if (std::fabs(next - x) <= close && (a_known || next != lo) && (b_known || next != hi)) return next;
      x = next;
    }
    return x;
  }

  // Atomic operation: the minimiser of the strongly
  // convex pair cost (Lemma 3) on (X/2, X), kept inside "one update, the quantiser's
  // shortest code" (1 bit for PQ; QSGD needs a sign bit and a level bit).  By slope: where the derivative is zero, half a dozen
  // evaluations from the size before on.  Else by golden-section search, 82 evaluations.
  double atomic_operation(double X, double z_r2, double size_before, bool by_slope) const {
    const double p_max = u_ / ((double)s_ + y_min_);
    double lo = 0.5 * X, hi = X - 1.0;
    if (hi > p_max) hi = p_max;
    if (lo < X - p_max) lo = X - p_max;
    if (!(hi > lo)) return 0.5 * X > p_max ? p_max : 0.5 * X;
    if (by_slope) {
      const double flat = flat_point(lo, hi, size_before, pair(X, z_r2));
      if (flat >= lo && flat <= hi) return flat;  // a number
    }
    const double g = 0.6180339887498949;
    double x1 = hi - g * (hi - lo), x2 = lo + g * (hi - lo);
    const Pair pr = pair(X, z_r2);
    double f1 = pair_cost(x1, pr), f2 = pair_cost(x2, pr);
    for (int it = 0; it < 80; ++it) {
      if (f1 <= f2) {
        hi = x2; x2 = x1; f2 = f1;
        x1 = hi - g * (hi - lo);
        f1 = pair_cost(x1, pr);
      } else {
        lo = x1; x1 = x2; f1 = f2;
        x2 = lo + g * (hi - lo);
        f2 = pair_cost(x2, pr);
      }
    }
    return 0.5 * (lo + hi);
  }

  // The plan for one k: SMO-style sweeps over the group sizes, then integer code lengths and refilled group sizes; returns gamma of
  // the integer plan.
  // `exact` = false: by slope where that can be.  The search would find a size only as well as the cost's rounding lets it: 5e-9 of
  // the size off as a rule, 7e-8 at most in a million k of random requests (4 to 3e7 coordinates, up to 60 bits each).  That
  // matters where u / size is next to a whole number, as it is for groups of whole sizes in small vectors, and where the sweeps
  // may end one earlier or later, which moves a size by little more than half a unit in either of its pairs.  *sure = false says so:
  // the result is then the least gamma that the search can end at.
  double solve(double k, bool exact, uint32_t* y, uint32_t* P, bool* sure) const {
    constexpr double kLoose = 2e-7;
    constexpr uint32_t kMostDoubts = 4;
    const bool by_slope = by_slope_ && !exact;
    double Pc[CVLC_MAX_CODED], nearest_stop = 1.0, largest = 0.0;
    for (uint32_t r = 0; r < R_; ++r) Pc[r] = k / (double)R_;
    for (int sweep = 0; sweep < 200; ++sweep) {
      double moved = 0.0, z_r2 = 0.0;
      for (uint32_t r = 1; r < R_; ++r) {
        const double X = Pc[r - 1] + Pc[r];
        const double Pr = atomic_operation(X, z_r2, Pc[r], by_slope);
        const double delta = std::fabs(Pr - Pc[r]);
        if (delta > moved) moved = delta;
        Pc[r] = Pr;
        Pc[r - 1] = X - Pr;
        z_r2 += Pc[r - 1];
      }
      nearest_stop = std::min(nearest_stop, std::fabs(moved - 0.5));
      if (moved < 0.5) break;
    }
    double bits[CVLC_MAX_CODED];  // a record's, rounded down
    uint32_t doubts[kMostDoubts], n_doubts = 0;
    for (uint32_t r = 0; r < R_; ++r) {
      bits[r] = std::floor(u_ / Pc[r]);
      largest = std::max(largest, Pc[r]);
    }
    const double stop = nearest_stop < kLoose * largest ? 1.25 : 0.0;
    for (uint32_t r = 0; r < R_ && by_slope; ++r) {
      const double t = u_ / Pc[r], length = t - (double)s_;  // lengths of 1 and 16 are the ends: the steps are at 2 .. 16
      if (!(length > 1.5 && length < 16.5 && std::fabs(t - std::round(t)) <= t * (kLoose + stop / Pc[r]))) continue;
      bits[r] = std::round(t);  // or one less
      if (n_doubts < kMostDoubts) doubts[n_doubts] = r;
      ++n_doubts;
    }
    *sure = n_doubts == 0;
    if (n_doubts > kMostDoubts) return -std::numeric_limits<double>::infinity();
    double least = integer_plan(bits, y, P);
    for (uint32_t choice = 1; choice < 1u << n_doubts; ++choice) {
      double other[CVLC_MAX_CODED];
      std::copy(bits, bits + R_, other);
      for (uint32_t i = 0; i < n_doubts; ++i)
        if (choice >> i & 1u) other[doubts[i]] -= 1.0;
      least = std::min(least, integer_plan(other, y, P));
    }
    return least;
  }

 private:
  // From the bits of a record: lengths clamped to the quantiser's range and non-increasing, groups refilled.
  double integer_plan(const double* bits, uint32_t* y, uint32_t* P) const {
    uint64_t room = d_;
    for (uint32_t r = 0; r < R_; ++r) {
      double yr = bits[r] - (double)s_;
      if (yr < y_min_) yr = y_min_;
      if (yr > 16.0) yr = 16.0;
      uint32_t yi = (uint32_t)yr;
      if (r > 0 && yi > y[r - 1]) yi = y[r - 1];
      uint64_t Pi = (uint64_t)(u_ / (double)(s_ + yi));
      if (Pi > room) Pi = room;
      y[r] = yi;
      P[r] = (uint32_t)Pi;
      room -= Pi;
    }
    return gamma_integer(d_, R_, P, y, alpha_, B_, quant_);
  }

  uint32_t d_, R_, s_;
  double u_;
  PowerLaw law_;
  ErrorModel err_;
  double alpha_, B_;
  uint32_t quant_;
  double y_min_;
  // Where the pairs' minima are found by slope: PQ (QSGD's error model has a kink) without scaling (the constant part of a scale factor
  // buries the minimum in rounding, so that the search decides the plan's last unit), and an exponent for which the pair cost is
  // convex and of a size that its rounding leaves alone: Lemma 3 assumes alpha < 0; below -10 the tail's energy vanishes beside the
  // head's and the two end up to a tenth of a size apart; near beta = 0, but for the limit itself, the power-law terms cancel (1e-6 of
  // a size at beta = 2e-5, 1e-2 at 2e-10).  Equal magnitudes fit an alpha of about 0 of either sign.
  bool by_slope_;
};

// CPUs the calling thread may run on.
int cpus() {
  cpu_set_t set;
  if (sched_getaffinity(0, sizeof set, &set) == 0) return CPU_COUNT(&set);
  return (int)std::thread::hardware_concurrency();  // more of them than the set can name
}

// Helper threads of all planner calls that run at the same time: as many as there are CPUs left besides the caller's,
// however many threads plan for their clients at once.
class Helpers {
 public:
  explicit Helpers(int most) {
    const int room = cpus() - 1;
    int running = running_.load();
    do {
      taken_ = std::max(0, std::min(most, room - running));
    } while (taken_ && !running_.compare_exchange_weak(running, running + taken_));
  }
  ~Helpers() { running_.fetch_sub(taken_); }
  Helpers(const Helpers&) = delete;
  Helpers& operator=(const Helpers&) = delete;
  int taken() const { return taken_; }

 private:
  static std::atomic<int> running_;
  int taken_;
};
std::atomic<int> Helpers::running_{0};

int plan_algorithm1(uint32_t d, uint64_t budget, uint32_t R, double alpha, float B, uint32_t quant,
                    cvlc_plan_t* out) {
  if (R < 1 || !std::isfinite(alpha) || quant > CVLC_QUANT_QSGD) return CVLC_ERR_ARG;
  plan_init(out, d, R, B);
  out->quant = quant;
  const int64_t b = group_share_bits(budget, R);
  if (b < (int64_t)kSegHeaderBits) return CVLC_ERR_BUDGET;
  const double u = (double)(b - kSegHeaderBits);
  const double k_min = (double)R;
  double k_max = (double)R * u / ((double)out->s + (quant == CVLC_QUANT_QSGD ? 2.0 : 1.0));
  if (k_max > (double)d) k_max = (double)d;
  if (k_max < k_min) return CVLC_ERR_BUDGET;
  const Algorithm1 alg(d, R, out->s, u, alpha, (double)B, quant);
  // Equidistant search over k.  The 128 searches know nothing of each other: they are shared out between up to 16 threads,
  // and the first of the best is taken as if they had been done in order (7 groups, 1.2 M coordinates: 424 us, with ten threads
  // 480; with golden-section searches alone, twelve times the evaluations, 2 007).  Then once more, exactly, those that by slope are
  // not sure and may be better than the best of the others: next to none (all that are not sure: one plan in ten took 100 us more).
  constexpr int kGrid = 128, kThreads = 16;
  struct Candidate {
    double gamma;
    bool sure;
    uint32_t y[CVLC_MAX_CODED], P[CVLC_MAX_CODED];
  };
  Candidate found[kGrid];
  int todo[kGrid], n_todo = kGrid;
  for (int g = 0; g < kGrid; ++g) todo[g] = g;
  auto search_all = [&](bool exact) {
    std::atomic<int> next{0};
    auto search = [&] {
      for (int i = next.fetch_add(1); i < n_todo; i = next.fetch_add(1)) {
        const int g = todo[i];
        const double k = k_min + (k_max - k_min) * (double)g / (double)(kGrid - 1);
        found[g].gamma = alg.solve(k, exact, found[g].y, found[g].P, &found[g].sure);
      }
    };
    const Helpers room(R > 1 ? std::min(kThreads, n_todo) - 1 : 0);  // one group: nothing to balance, microseconds in all
    std::thread helpers[kThreads - 1];
    try {
      for (int t = 0; t < room.taken(); ++t) helpers[t] = std::thread(search);
    } catch (...) {
      // no more threads (or no memory for them) to be had: those that run and this one do the work
    }
    search();
    for (std::thread& t : helpers)
      if (t.joinable()) t.join();
  };
  search_all(false);
  double best_sure = std::numeric_limits<double>::infinity();
  for (const Candidate& c : found)
    if (c.sure && c.gamma < best_sure) best_sure = c.gamma;
  n_todo = 0;
  for (int g = 0; g < kGrid; ++g)
    if (!found[g].sure && !(found[g].gamma > best_sure)) todo[n_todo++] = g;
  if (n_todo) search_all(true);
  double best = std::numeric_limits<double>::infinity();
  for (const Candidate& c : found) {
    if (c.gamma < best) {
      best = c.gamma;
      for (uint32_t r = 0; r < R; ++r) {
        out->code_len[r] = c.y[r];
        out->count[r] = c.P[r];
      }
    }
  }
  if (!(best < std::numeric_limits<double>::infinity())) return CVLC_ERR_BUDGET;
  out->total_bits = cvlc_plan_total_bits(out);
  if (out->total_bits > budget) return CVLC_ERR_BUDGET;
  return cvlc_plan_validate(out);
}

}  // namespace

extern "C" {

uint32_t cvlc_position_bits(uint32_t d) { return cvlc::position_bits(d); }

uint64_t cvlc_plan_total_bits(const cvlc_plan_t* p) {
  if (!p) return 0;
  uint64_t words = cvlc::kGlobalHeaderWords + (uint64_t)cvlc::kSegHeaderWords * p->n_coded;
  for (uint32_t r = 0; r < p->n_coded && r < CVLC_MAX_CODED; ++r)
    words += cvlc::payload_words(p->count[r], p->s + p->code_len[r]);
  return 32u * words;
}

int cvlc_plan_validate(const cvlc_plan_t* p) {
  if (!p) return CVLC_ERR_ARG;
  if (p->d < 1 || p->d > 0x7FFFFFFFu) return CVLC_ERR_PLAN;
  if (p->n_coded > CVLC_MAX_CODED) return CVLC_ERR_PLAN;
  if (p->s != cvlc::position_bits(p->d)) return CVLC_ERR_PLAN;
  if (p->quant > CVLC_QUANT_QSGD) return CVLC_ERR_PLAN;
  if (!(p->B > 0.0f) || !std::isfinite(p->B)) return CVLC_ERR_PLAN;
  uint64_t k = 0;
  for (uint32_t r = 0; r < p->n_coded; ++r) {
    if (!cvlc::code_len_supported(p->code_len[r])) return CVLC_ERR_PLAN;
    if (p->quant == CVLC_QUANT_QSGD && p->code_len[r] < 2) return CVLC_ERR_PLAN;  // a sign bit and a level bit
    if (r > 0 && p->code_len[r] > p->code_len[r - 1]) return CVLC_ERR_PLAN;
    k += p->count[r];
  }
  if (k > p->d) return CVLC_ERR_PLAN;
  if (p->total_bits != cvlc_plan_total_bits(p)) return CVLC_ERR_PLAN;
  return CVLC_OK;
}

double cvlc_plan_gamma(const cvlc_plan_t* p, double alpha) {
  if (!p || p->n_coded > CVLC_MAX_CODED) return std::numeric_limits<double>::quiet_NaN();
  return gamma_integer(p->d, p->n_coded, p->count, p->code_len, alpha, (double)p->B, p->quant);
}

double cvlc_plan_next_scale(const cvlc_plan_t* plan) {
  double worst = 0.0;
  if (plan) {
    const uint32_t R = plan->n_coded < CVLC_MAX_CODED ? plan->n_coded : CVLC_MAX_CODED;
    for (uint32_t r = 0; r < R; ++r) {
      const uint32_t y = plan->code_len[r];
      if (y == 0 || y >= 32 || plan->count[r] == 0) continue;  // raw values carry no quantisation error
      const double Q = plan->quant == CVLC_QUANT_QSGD ? qsgd_error((double)plan->count[r], (double)y)
                                                      : pq_error((double)plan->count[r], (double)y);
      if (Q > worst) worst = Q;
    }
  }
  return worst + 1.0;
}

double cvlc_stats_gamma(const cvlc_seg_stats_t* stats, uint32_t n_coded) {
  if (!stats || n_coded > CVLC_MAX_CODED) return 0.0;
  double err = 0.0, all = 0.0;
  for (uint32_t r = 0; r <= n_coded; ++r) {
    err += stats[r].errsq;
    all += stats[r].sumsq;
  }
  return all > 0.0 ? err / all : 0.0;
}

size_t cvlc_stream_capacity(const cvlc_plan_t* p) { return p ? (size_t)(p->total_bits / 8u) : 0; }

int cvlc_plan(uint32_t d, uint64_t budget_bits, uint32_t n_coded, const uint32_t* code_len,
              const double* fractions, double alpha, float B, cvlc_plan_t* out) {
  if (!out || d < 1 || d > 0x7FFFFFFFu || n_coded > CVLC_MAX_CODED) return CVLC_ERR_ARG;
  if (!(B > 0.0f) || !std::isfinite(B)) return CVLC_ERR_ARG;
  if (fractions) {
    if (!code_len) return CVLC_ERR_ARG;
    return plan_from_fractions(d, n_coded, code_len, fractions, B, out);
  }
  if (code_len) return plan_from_budget(d, budget_bits, n_coded, code_len, B, out);
  return plan_algorithm1(d, budget_bits, n_coded, alpha, B, CVLC_QUANT_PQ, out);
}

int cvlc_plan_algorithm1(uint32_t d, uint64_t budget_bits, uint32_t n_coded, double alpha, float B, uint32_t quant,
                         cvlc_plan_t* out) {
  if (!out || d < 1 || d > 0x7FFFFFFFu || n_coded > CVLC_MAX_CODED) return CVLC_ERR_ARG;
  if (!(B > 0.0f) || !std::isfinite(B)) return CVLC_ERR_ARG;
  return plan_algorithm1(d, budget_bits, n_coded, alpha, B, quant, out);
}

const char* cvlc_status_string(int status) {
  switch (status) {
    case CVLC_OK: return "ok";
    case CVLC_ERR_ARG: return "bad argument";
    case CVLC_ERR_PLAN: return "invalid plan";
    case CVLC_ERR_BUDGET: return "budget too small";
    case CVLC_ERR_CAPACITY: return "buffer too small";
    case CVLC_ERR_NONFINITE: return "non-finite input";
    case CVLC_ERR_STREAM: return "malformed stream";
    case CVLC_ERR_DEVICE: return "HIP call failed";
    default: return "unknown status";
  }
}

}  // extern "C"

namespace cvlc {
int hip_check(hipError_t e) { return e == hipSuccess ? CVLC_OK : CVLC_ERR_DEVICE; }

namespace {
struct Bracket {
  int stage;
  hipEvent_t begin, end;
};
bool g_profiling = false;
uint32_t g_stage_mask = 0;
std::vector<Bracket> g_brackets;
}  // namespace

void profile_mark(int stage, bool begin, hipStream_t stream) {
  if (!g_profiling || !((g_stage_mask >> stage) & 1u)) return;
  if (begin) {
    Bracket b{stage, nullptr, nullptr};
    if (hipEventCreate(&b.begin) != hipSuccess || hipEventCreate(&b.end) != hipSuccess) return;
    (void)hipEventRecord(b.begin, stream);
    g_brackets.push_back(b);
  } else {
    for (size_t i = g_brackets.size(); i-- > 0;)
      if (g_brackets[i].stage == stage) {
        (void)hipEventRecord(g_brackets[i].end, stream);
        break;
      }
  }
}
}  // namespace cvlc

extern "C" {

int cvlc_profile_start(uint32_t stage_mask) {
  if (cvlc::g_profiling) return CVLC_ERR_ARG;
  cvlc::g_stage_mask = stage_mask;
  cvlc::g_brackets.clear();
  cvlc::g_profiling = true;
  return CVLC_OK;
}

int cvlc_profile_stop(float* ms_per_stage, uint32_t* brackets_per_stage) {
  if (!cvlc::g_profiling || !ms_per_stage || !brackets_per_stage) return CVLC_ERR_ARG;
  cvlc::g_profiling = false;
  for (int i = 0; i < CVLC_PROFILE_STAGES; ++i) { ms_per_stage[i] = 0.0f; brackets_per_stage[i] = 0; }
  int rc = CVLC_OK;
  for (auto& b : cvlc::g_brackets) {
    float ms = 0.0f;
    if (hipEventSynchronize(b.end) == hipSuccess && hipEventElapsedTime(&ms, b.begin, b.end) == hipSuccess) {
      ms_per_stage[b.stage] += ms;
      brackets_per_stage[b.stage] += 1;
    } else {
      rc = CVLC_ERR_DEVICE;
    }
    (void)hipEventDestroy(b.begin);
    (void)hipEventDestroy(b.end);
  }
  cvlc::g_brackets.clear();
  return rc;
}

}  // extern "C"
