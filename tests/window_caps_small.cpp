// The window replay of window_caps.cpp for the forward's 64 x 4 tile, which
// small outputs take.
#define main window_caps_main
#include "window_caps.cpp"
#undef main

int main() {
  std::mt19937_64 rng(5);
  const int sizes[][2] = {{256, 256}, {64, 48}, {4, 4}, {96, 136}};
  for (auto& sz : sizes)
    for (int T : {8, 16, 64})
      for (double s : {1.0, 1.25, 2.0, 3.0}) {
        const Geometry g = geometry(sz[0], sz[1], T, s);
        for (int field = 0; field < 3; ++field) {
          std::vector<float> mo((size_t)g.TY * g.TX * 2);
          for (auto& v : mo)
            v = field == 0 ? (float)((int)(rng() % 81) - 40) * 0.25f
                           : (field == 1 ? (rng() & 1 ? 400.f : -400.f) : (rng() % 5 ? 3.7f : NAN));
          if (!check_tiles<4>(g, mo)) return 1;
        }
      }
  printf("OK %lld pixels\n", g_checked);
  return 0;
}
