// k_topk_choose, workgroup by workgroup, its wavefronts in several orders (emulated_wavefronts.h): one tensor of a ring, whose drifts, key
// codes and counts are made here, and the selection that they have to give.  Arguments: elements, K, what the keys are like (see
// drifts()), whether the ring has key codes to go by.  Prints what is wrong.
#include "emulated_wavefronts.h"

#include "kernels_choose.hip"        // (without its launch, and with its LDS as emu::dynamic_lds: the test writes that file)

#include <random>
#include <string>

using namespace evg;

// `ties`: how many have the K-th largest magnitude, the K-th among them somewhere in the middle, so that some of them lose.  `near`:
// others that differ from it in the last bits only.
static std::vector<float> drifts(uint32_t n, uint32_t K, uint32_t ties, uint32_t near, uint32_t seed) {
  std::mt19937 gen(seed);
  std::vector<float> d(n);
  for (float& v : d) v = std::exp2(-8.0f + (float)(gen() >> 8) * 0x1p-24f * 4.0f) * (gen() & 1 ? 1.0f : -1.0f);
  std::vector<uint32_t> by(n);
  for (uint32_t i = 0; i < n; ++i) by[i] = i;
  std::sort(by.begin(), by.end(), [&](uint32_t a, uint32_t b) { return std::fabs(d[a]) > std::fabs(d[b]); });
  const uint32_t first = K > ties / 2 ? K - ties / 2 : 0, bits = __float_as_uint(std::fabs(d[by[K - 1]])) | 3u;
  for (uint32_t i = first; i < std::min(n, first + ties); ++i) d[by[i]] = __uint_as_float(bits);
  for (uint32_t i = std::min(n, first + ties), q = 0; q < near && i < n; ++i, ++q) d[by[i]] = __uint_as_float(bits - 1 - q % 3);
  return d;
}

int main(int argc, char** argv) {
  if (argc != 6) return 2;
  const uint32_t n = std::atoi(argv[1]), K = std::atoi(argv[2]), ties = std::atoi(argv[3]), near = std::atoi(argv[4]);
  const bool codes = std::atoi(argv[5]) != 0;
  constexpr uint32_t P = 3, r = 0, SW = 2, chunk = SW * 1024;
  const uint32_t C = (n + chunk - 1) / chunk, Npad = (n + 63) / 64 * 64, ngroups = (n + 255) / 256;

  const std::vector<float> d = drifts(n, K, ties, near, n + K);
  std::vector<uint32_t> key(n), by(n);
  for (uint32_t j = 0; j < n; ++j) { key[j] = __float_as_uint(std::fabs(d[j])); by[j] = j; }
  std::stable_sort(by.begin(), by.end(), [&](uint32_t a, uint32_t b) { return key[a] > key[b]; });
  const uint32_t t = key[by[K - 1]];
  uint32_t above = 0, equal = 0;
  for (uint32_t k : key) { above += k > t; equal += k == t; }

  std::vector<float> x(P * Npad), xhat(P * Npad);
  for (uint32_t j = 0; j < n; ++j) x[r * Npad + j] = d[j];
  std::vector<uint8_t> code(P * Npad + 16);
  const uint32_t q = t >> kFineBits, anchor = !codes ? kNoAnchor : q > 128 ? (q - 128) / kPerCoarse * kPerCoarse : 0;

  std::vector<double> partials(P * C * SW, 1.0);
  std::vector<float> delta(P), last_norm(P), before(P), slope(P);
  std::vector<int32_t> last_event(P);
  std::vector<uint8_t> valid_l(4), valid_r(4), fired(4), tie(4);
  std::vector<uint32_t> ev_full(P), ev_topk(P), near_cnt(P), nonfinite(P), slope_cnt(P), not_staged(1), prefix(P), krem(P), cut(P), anchors(P, anchor);
  std::vector<uint32_t> group(P * C * SW * 4);
  std::vector<uint2> chunk_before(P * C);
  IterState it{};
  Tables T{};
  T.x = x.data(); T.xhat = xhat.data(); T.codes = code.data(); T.partials = partials.data();
  T.delta = T.delta_out = delta.data(); T.last_norm = last_norm.data(); T.delta_before = before.data();
  T.last_event = T.last_event_out = last_event.data();
  T.valid_l = valid_l.data(); T.valid_r = valid_r.data(); T.fired = fired.data(); T.near_tie = tie.data();
  T.ev_full = ev_full.data(); T.ev_topk = ev_topk.data(); T.near_cnt = near_cnt.data(); T.nonfinite_cnt = nonfinite.data();
  T.slope_hist = slope.data(); T.slope_cnt = slope_cnt.data(); T.not_staged = not_staged.data();
  T.sel_prefix = prefix.data(); T.sel_krem = krem.data(); T.sel_cut = cut.data(); T.anchor = anchors.data();
  T.group = group.data(); T.chunk_before = chunk_before.data(); T.it = &it;
  T.P = P; T.L = 1; T.C = C; T.S = P; T.SW = SW; T.fine = 1; T.hist_len = 1; T.Npad = Npad;
  StepArgs A{};
  A.k = 5;
  A.topk_on = 1;
  const ChooseDesc desc{0, 0, n, K, 0, C, 0, C * SW};
  const uint32_t cap = n <= 327680 ? 4096u : 12288u;
  int wrong = 0;
  for (int order = 0; order < 4; ++order) {
    std::vector<uint32_t> hist(P * kHistBins);
    for (uint32_t j = 0; j < n; ++j) {
      const uint32_t k = key[j] >> kFineBits, c = anchor == kNoAnchor || k < anchor ? 0 : std::min(k - anchor, 255u);
      code[r * Npad + j] = (uint8_t)c;
      if (c >= kFirstCode) ++hist[r * kHistBins + j % 8 * kCodeStride + std::min(c - kFirstCode, kCodeBins)];
    }
    T.hist = hist.data();
    last_event.assign(P, 0);
    delta.assign(P, 0.0f);
    anchors.assign(P, anchor);
    group.assign(group.size(), 0xABABABAB);
    chunk_before.assign(chunk_before.size(), uint2{0xABABABAB, 0xABABABAB});
    not_staged[0] = 0;
    emu::dynamic_lds.assign(ngroups + 2 * cap, 0xCDCDCDCD);
    emu::block_idx = {0, r, 1};
    emu::run(kWide, order < 2 ? (emu::Order)order : emu::Order::kRandom, 77u + order, [&] { k_topk_choose(&desc, n > 256, ngroups, cap, A, T); });
    // who wins: all above the threshold, of those equal to it the first `ties`
    const uint32_t wins = K - above;
    if (fired[r] != 2 || prefix[r] != t || krem[r] != wins)
      std::printf("order %d: code %u threshold %08x ties %u, not %08x %u\n", order, fired[r], prefix[r], krem[r], t, wins), wrong = 1;
    uint32_t sent = 0;
    for (uint32_t j = 0; j < n; ++j) sent += key[j] == t && j <= cut[r];
    if (sent != wins) std::printf("order %d: %u of the equal ones up to element %u, not %u\n", order, sent, cut[r], wins), wrong = 1;
    uint32_t a = 0, e = 0, bad = 0;
    for (uint32_t g = 0; g < ngroups; ++g) {
      const uint2 c = chunk_before[r * C + g / (SW * 4)];
      const uint32_t in = group[r * C * SW * 4 + g];
      bad += c.x + (in & 0xFFFF) != a || c.y + (in >> 16) != e;
      for (uint32_t j = g * 256; j < std::min(n, g * 256 + 256); ++j) { a += key[j] > t; e += key[j] == t; }
    }
    if (bad) std::printf("order %d: places of %u groups\n", order, bad), wrong = 1;
    if (it.iters != (uint64_t)order + 1) std::printf("order %d: %u steps booked\n", order, (unsigned)it.iters), wrong = 1;
  }
  if (!wrong) std::printf("ok equal %u staged %d\n", equal, not_staged[0] == 0);
  return 0;
}
