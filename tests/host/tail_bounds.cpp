// Runs fold_tail_block on host threads, a workgroup of `threads` at a time, with its input, its
// output and its LDS array each ending at a guard page: an access out of range ends the
// process with a signal.  Outputs are compared with eq. (3)'s fold written out.
//   tail_bounds F threads   (n = q + F qubits, q = 6: the sizes of the batch's tail stage)
#include <cstdio>
#include <thread>
#include <vector>

#include "guarded.hpp"
#include "lre_tile.hpp"

using namespace lre;

template <int F, class Acc, Out MODE>
int run(int threads) {
  using G = FoldTailGeom<F>;
  constexpr int q = 6, n = q + F;
  const int64_t L = (int64_t)1 << (2 * q), rows = ipow3(F), cols = 1 << F;
  Acc* in = guarded<Acc>((size_t)(rows * cols * L));
  double* out = guarded<double>((size_t)(L << (2 * F)));
  Acc* mid = guarded<Acc>(F > 2 ? G::SUB * 16 * G::COLS : 1);
  for (int64_t i = 0; i < rows * cols * L; ++i) in[i] = (Acc)((i * 2654435761u >> 7) % 1000);
  const int64_t blocks = L / G::COLS, shots = MODE == Out::CoefUniform ? 7 : 0;
  for (int64_t blk : {(int64_t)0, blocks / 2, blocks - 1}) {
    std::barrier<> bar(threads);
    host_barrier = &bar;
    std::vector<std::thread> group;
    for (int t = 0; t < threads; ++t)
      group.emplace_back([=] { fold_tail_block<F, Acc, Acc, MODE>(in, out, n, F, q, shots, blk, t, mid); });
    for (auto& t : group) t.join();
    for (int a = 0; a < (1 << (2 * F)); ++a)
      for (int64_t c = blk * G::COLS; c < (blk + 1) * G::COLS; ++c) {
        double want = 0;
        int w = 0;
        for (uint64_t v = (uint64_t)a << (2 * q) | (uint64_t)c; v; v >>= 2) w += (v & 3) != 0;
        for (int64_t b = 0; b < rows; ++b)
          for (int64_t s = 0; s < cols; ++s) {
            int sign = 1, p3 = 1;
            for (int k = 0; k < F; ++k, p3 *= 3) {
              const int letter = a >> (2 * k) & 3;
              if (letter == 0) continue;
              if (b / p3 % 3 != letter - 1) sign = 0;
              else if (s >> k & 1) sign = -sign;
            }
            want += sign * (double)in[(b * cols + s) * L + c];
          }
        want /= std::pow(3.0, n - w) * (shots ? shots : 1);
        if (out[a * L + c] != want) {
          std::printf("F %d block %ld code %d column %ld: %.17g, not %.17g\n", F, (long)blk, a, (long)c, out[a * L + c], want);
          return 1;
        }
      }
  }
  return 0;
}

template <int F>
int both(int threads) {
  return run<F, uint32_t, Out::CoefUniform>(threads) | run<F, double, Out::CoefPerBasis>(threads);
}

int main(int argc, char** argv) {
  if (argc != 3) return 2;
  const int threads = std::atoi(argv[2]);
  switch (std::atoi(argv[1])) {
    case 1: return both<1>(threads);
    case 2: return both<2>(threads);
    case 3: return both<3>(threads);
    case 4: return both<4>(threads);
  }
  return 2;
}
