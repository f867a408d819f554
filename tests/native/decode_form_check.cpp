// Host side of the small-batch tiles' forms (csrc/decode_form.h).
//
// Without arguments: checks that each staged form's workgroups fit on a CU as
// many as it says, that P's form beside D leaves a D tile's LDS however many of its
// workgroups a CU holds, and that the forms beside the other phase depend on
// nothing else.  With "form E E_loc k T n_tiles": prints the form of a launch.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>

#include "decode_form.h"

using namespace moepd;

int main(int argc, char** argv) {
  if (argc == 7 && !std::strcmp(argv[1], "form")) {
    const int E = std::atoi(argv[2]), e_loc = std::atoi(argv[3]), k = std::atoi(argv[4]), T = std::atoi(argv[5]);
    std::printf("%d\n", (int)decode_form(decode_m_tiles(E, e_loc, k, T) * std::atoi(argv[6]), Beside::kNone));
    return 0;
  }
  int bad = 0;
  const int units = kLdsPerCu / kLdsUnit;
  for (int mx = 0; mx < 2; ++mx)
    for (int form : {kDecodeFour, kDecodeSix, kDecodeEight}) {
      const int fit = units / lds_units(decode_lds(form, mx));
      if (fit != form) {
        std::printf("%s form of %d per CU: %d bytes, %d fit\n", mx ? "FP8" : "bf16", form, decode_lds(form, mx), fit);
        ++bad;
      }
    }
  const auto room = [](double tiles) { return decode_form(tiles, Beside::kLeaveRoom); };
  const auto fit = [](double tiles) { return decode_form(tiles, Beside::kFit); };
  for (int mx = 0; mx < 2; ++mx)
    for (double tiles : {1.0, 100.0, 1024.0, 1025.0, 1536.0, 2048.0, 2560.0, 1e5}) {
      const int p = lds_units(decode_lds(room(tiles), mx)), d = lds_units(decode_lds(fit(tiles), mx));
      const int left = units - units / p * p;
      if (left < d) {
        std::printf("%s, %g tiles: P's leave %d units of LDS, D's tile takes %d\n", mx ? "FP8" : "bf16", tiles, left, d);
        ++bad;
      }
    }
  if (bad) return 1;
  std::printf("ok\n");
  return 0;
}
