// Host-side check of the packed list entries of the families with two
// dependent axes (RAY3D 12 bytes, SIM2D 16 bytes) and of the one-word PLANE3D
// entry cut 9 | 9 | 14 bits: every value inside the limits round-trips
// exactly, one field beyond its limit is flagged.
#include "../../paper_2107_11810_amd/csrc/gv_device.h"
#include <cstdio>
#include <cstdlib>

static int fails = 0;
#define CHECK(c)                                              \
  do {                                                        \
    if (!(c)) {                                               \
      std::printf("FAIL %s:%d %s\n", __FILE__, __LINE__, #c); \
      fails++;                                                \
    }                                                         \
  } while (0)

template <int FAM> static bool same(const LinS& a, const LinS& b) {
  bool r = a.w == b.w && a.tag == b.tag && a.F[0] == b.F[0] && a.F[1] == b.F[1];
  for (int q = 0; q < 2; q++)
    for (int p = 0; p < 2; p++) r = r && a.K[q][p] == b.K[q][p];
  return r;
}

template <int FAM, typename E> static void check(int32_t wmax) {
  const int32_t v[] = {0, 1, -1, 2, -2, 12345, -12345, GV_L2_MAX - 1, GV_L2_MAX, -GV_L2_MAX};
  const int32_t ws[] = {1, 2, 65536, wmax - 1, wmax};
  for (int32_t a : v)
    for (int32_t b : v)
      for (int32_t f : v)
        for (int32_t w : ws)
          for (int32_t tag = 0; tag < (FAM == FAM_RAY3D ? 3 : 1); tag++) {
            LinS s = lin_zero<FAM>();
            s.K[0][0] = a;
            s.K[1][0] = b;
            if (FAM == FAM_SIM2D) {
              s.K[0][1] = b;
              s.K[1][1] = -a;
            }
            s.F[0] = f;
            s.F[1] = -b;
            s.w = w;
            s.tag = tag;
            bool ok = true;
            const E e = store_ent<FAM, E>(s, ok);
            CHECK(ok);
            CHECK(same<FAM>(load_ent<FAM>(e), s));
          }
  const int32_t out[] = {GV_L2_MAX + 1, -GV_L2_MAX - 1};
  for (int32_t x : out)
    for (int k = 0; k < 6; k++) {
      if (FAM == FAM_RAY3D && (k == 1 || k == 3)) continue;  // (one parameter axis)
      LinS s = lin_zero<FAM>();
      s.w = 1;
      (k < 4 ? s.K[k / 2][k % 2] : s.F[k - 4]) = x;
      bool ok = true;
      (void)store_ent<FAM, E>(s, ok);
      CHECK(!ok);
      ok = false;  // a flag once cleared stays cleared
      (void)store_ent<FAM, E>(lin_zero<FAM>(), ok);
      CHECK(!ok);
    }
}

int main() {
  static_assert(sizeof(EntR3p) == 12 && sizeof(EntS2p) == 16, "packed entry sizes");
  check<FAM_RAY3D, EntR3p>(GV_R3_WMAX);
  check<FAM_SIM2D, EntS2p>(0x7fffffff);
  static_assert(sizeof(EntP3v) == 4, "one word");
  for (int32_t K1 = -GV_P3V_KMAX - 1; K1 <= GV_P3V_KMAX + 1; K1++)
    for (int32_t K2 : {0, 1, -1, GV_P3V_KMAX, -GV_P3V_KMAX, GV_P3V_KMAX + 1, -GV_P3V_KMAX - 1})
      for (int32_t F : {0, 1, -1, 4097, GV_P3V_FMAX, -GV_P3V_FMAX, GV_P3V_FMAX + 1, -GV_P3V_FMAX - 1}) {
        LinS s = lin_zero<FAM_PLANE3D>();
        s.K[0][0] = K1;
        s.K[0][1] = K2;
        s.F[0] = F;
        s.w = 1;
        const bool in = abs(K1) <= GV_P3V_KMAX && abs(K2) <= GV_P3V_KMAX && abs(F) <= GV_P3V_FMAX;
        bool ok = true;
        const EntP3v e = store_ent<FAM_PLANE3D, EntP3v>(s, ok);
        CHECK(ok == in);
        if (in) CHECK(same<FAM_PLANE3D>(load_ent<FAM_PLANE3D>(e), s));
      }
  {
    LinS s = lin_zero<FAM_RAY3D>();
    s.w = GV_R3_WMAX + 1;
    bool ok = true;
    (void)store_ent<FAM_RAY3D, EntR3p>(s, ok);
    CHECK(!ok);
  }
  // round half to even of x / 2
  for (int32_t x = -4099; x <= 4099; x++) {
    int32_t q = (x - (x & 1)) / 2;  // floor
    if ((x & 1) && (q & 1)) q++;
    CHECK(rne_half(x) == q);
  }
  std::printf(fails ? "%d FAILURES\n" : "OK\n", fails);
  return fails ? 1 : 0;
}
