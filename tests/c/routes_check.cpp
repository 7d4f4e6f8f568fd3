// Prints the dispatch rules' answers, one line for each query line of stdin:
//   read io state d_ff d_model count context_bytes                -> direct waves leaf nt
//   write io state d_ff d_model count chunk token context_bytes   -> kernel read_first wn nt
//   adapter slices chunk count rank                               -> tiles of evidence rows per block
//   gemm count mt ntl                                             -> 1 if every tile is dealt once, then tiles of each XCD
#include <cstdio>
#include <iostream>
#include <string>
#include <vector>

#include "rwttt_routes.h"

using namespace rwttt;

static const char* name(WriteKernel k) {
  switch (k) {
    case WriteKernel::f32: return "f32";
    case WriteKernel::rows_token: return "rows_token";
    case WriteKernel::stream: return "stream";
    case WriteKernel::rows: return "rows";
    case WriteKernel::gemm: return "gemm";
  }
  return "?";
}

int main() {
  std::string what, io, state;
  while (std::cin >> what) {
    if (what == "read") {
      int d_ff, d_model, count;
      size_t context;
      std::cin >> io >> state >> d_ff >> d_model >> count >> context;
      const ReadRoute r = read_route(io == "bf16", state == "bf16", d_ff, d_model, count, context);
      std::printf("%d %d %d %d\n", r.direct, r.waves, r.leaf, r.nt);
    } else if (what == "write") {
      int d_ff, d_model, count, chunk, token;
      size_t context;
      std::cin >> io >> state >> d_ff >> d_model >> count >> chunk >> token >> context;
      const WriteRoute r =
          write_route(io == "bf16", state == "bf16", d_ff, d_model, count, chunk, token != 0, context);
      std::printf("%s %d %d %d\n", name(r.kernel), r.read_first, r.wn, r.nt);
    } else if (what == "adapter") {
      int slices, chunk, count, rank;
      std::cin >> slices >> chunk >> count >> rank;
      std::printf("%d\n", adapter_pq_tiles(slices, chunk, count, rank));
    } else if (what == "gemm") {
      int count, mt, ntl;
      std::cin >> count >> mt >> ntl;
      std::vector<int> seen(size_t(count) * mt * ntl);
      int xcd[8] = {0};
      const unsigned blocks = gemm_blocks(count, mt, ntl);
      for (unsigned i = 0; i < blocks; ++i) {
        const GemmTile t = gemm_tile(i, mt, ntl);
        if (t.b < 0 || t.b >= count || t.mt < 0 || t.mt >= mt || t.nt < 0 || t.nt >= ntl) continue;
        ++seen[(size_t(t.b) * mt + t.mt) * ntl + t.nt];
        ++xcd[i & 7];
      }
      bool once = true;
      for (int s : seen) once = once && s == 1;
      std::printf("%d", once);
      for (int x : xcd) std::printf(" %d", x);
      std::printf("\n");
    } else {
      return 1;
    }
  }
  return 0;
}
