// Host side of the small-batch tiles' forms (csrc/decode_form.h).
//
// Without arguments: checks that each staged form's workgroups fit on a CU as
// many as it says.  With "form E E_loc k T n_tiles": prints the form of a launch.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>

#include "decode_form.h"

using namespace moepd;

int main(int argc, char** argv) {
  if (argc == 7 && !std::strcmp(argv[1], "form")) {
    const int E = std::atoi(argv[2]), e_loc = std::atoi(argv[3]), k = std::atoi(argv[4]), T = std::atoi(argv[5]);
    std::printf("%d\n", (int)decode_form(decode_m_tiles(E, e_loc, k, T) * std::atoi(argv[6])));
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
  if (bad) return 1;
  std::printf("ok\n");
  return 0;
}
