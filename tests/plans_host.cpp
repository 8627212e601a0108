// The host's choice of a launch, for tests that ask which variant of a kernel their shapes take.
#include "gemm_direct_plan.hpp"
#include "kron_tile_plan.hpp"

using namespace tc355;

// second, wide, nb, lsp, blocks of I, blocks of J, tiles per wavefront, stages, workgroups that walk over them; 0 where the
// kernel does not take the layer
extern "C" int kron(int64_t B, int64_t I, int64_t K, int64_t J, int64_t L, int cus, int64_t* out) {
  KronTilePlan p{};
  if (!choose_kron_tile(B, I, K, J, L, cus, &p)) return 0;
  const int64_t i_blocks = p.second ? p.jblocks : p.iblocks, j_blocks = p.second ? p.iblocks : p.jblocks;  // (extents are exchanged)
  const int64_t plan[9] = {p.second, p.wide, p.nb, p.lsp, i_blocks, j_blocks, p.tj, p.groups, kron_tile_workgroups(p, cus)};
  for (int i = 0; i < 9; i++) out[i] = plan[i];
  return 1;
}

extern "C" void direct(int64_t N, int64_t M, int64_t K, int size, int cus, int* out) {
  const GemmDirectVariant& v = GD_VARIANTS[choose_gemm_direct(N, M, K, size, cus)];
  out[0] = v.rt;
  out[1] = v.ct;
  out[2] = v.nw;
}
