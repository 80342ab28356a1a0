// The kernel that the network's launchers choose, for shapes read from stdin:
//   conv <mode> <up> <batch> <side> <cin> <cout> <cout8>  -> th cw mt np
//   wgrad <batch> <side> <cin> <cout8> <taps>             -> columns small
#include <iostream>
#include <string>

#include "cnn.hpp"

int main() {
  using namespace lshom::cnn;
  std::string what;
  while (std::cin >> what) {
    if (what == "conv") {
      ConvArgs a{};
      std::cin >> a.mode >> a.up >> a.B >> a.Ho >> a.C0 >> a.N >> a.Np;
      a.Wo = a.Ho;
      const ConvVariant v = conv_variant(a);
      std::cout << v.th << ' ' << v.cw << ' ' << v.mt << ' ' << v.np << '\n';
    } else {
      WgradArgs a{};
      std::cin >> a.B >> a.Ho >> a.C0 >> a.Np >> a.taps;
      a.Wo = a.Ho;
      a.rows = a.taps * a.C0 + 1;
      const WgradVariant v = wgrad_variant(a, wgrad_splits((long long)a.B * a.Ho * a.Wo));
      std::cout << v.columns << ' ' << (v.small ? 1 : 0) << '\n';
    }
  }
}
