// FP64 links and corners of a lattice whose matrix slabs pass 4 GiB (64^3 x
// 128: 33.5 million sites), stored on the host by the functions of the setup
// kernels into memory that is reserved but only touched where they store.
// Prints, per store, whether every entry is where the 64-bit readers look for
// it (matrix slab k of the site at element k Vp + i) and nothing else changed
// there.
#include <sys/mman.h>

#include <cstdio>

#include "../paper_1312_3265_amd/csrc/common.h"

using namespace lq;

int main() {
  const int V = 64 * 64 * 64 * 128, Vp = (V + 63) / 64 * 64 + 64;
  const size_t bytes = (size_t)8 * 9 * Vp * sizeof(double2);
  void* mem = mmap(nullptr, bytes, PROT_READ | PROT_WRITE,
                   MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (mem == MAP_FAILED) return 2;
  double2* u = (double2*)mem;
  const int sites[] = {0, 1, 511, 512, 513, V / 2, V - 1};
  for (int corner = 0; corner < 2; ++corner) {
    const int nrec = corner ? 8 : 4;
    bool ok = true;
    for (int rec = 0; rec < nrec; ++rec)
      for (int i : sites) {
        double2 m[9];
        for (int k = 0; k < 9; ++k) m[k] = make_double2(1 + k + 10 * rec, i + 1);
        if (corner) store_corner<F64>(u, Vp, rec, i, m);
        else store_link<F64, 18>(u, Vp, rec, i, m);
      }
    for (int rec = 0; rec < nrec; ++rec)
      for (int i : sites)
        for (int k = 0; k < 9; ++k) {
          const double2 z = u[(size_t)(rec * 9 + k) * Vp + i];
          ok = ok && z.x == 1 + k + 10 * rec && z.y == i + 1;
        }
    std::printf("%s %s\n", corner ? "corners" : "links", ok ? "ok" : "wrong");
  }
  return 0;
}
