// Replays how the block kernels cut a unit's key stream, with the library's own plans and StreamCut, and prints
// what the shares ask of the slot tables.  One case a line on stdin:
//   S Hkv Hq C V ld max_L full  L nsel[0] .. nsel[V-1]
// and for each:  forward nW, most tiles of a share (each piece's last one padded), record slots used beyond
// nW + branches - 1, entries left out or taken twice;  backward nW, most entries of a piece, entries left out or
// taken twice, tiles of the longest stream the plan admits.
#include <cstdio>
#include <vector>

#include "bd_kernels.hpp"
#include "attn_tile.hpp"

template <class Cut>
static void replay(const std::vector<int>& len, int V, int nW, int64_t& tiles, int64_t& piece, int64_t& wrong, int64_t& recs) {
  int64_t total = 0, vt = 0;
  for (size_t b = 0; b < len.size(); ++b) {
    total += len[b];
    if ((int)b < V) vt += len[b];
  }
  const Cut cut((int)vt, (int)total, nW);
  tiles = piece = wrong = recs = 0;
  int64_t at = 0;
  for (int w = 0; w < nW; ++w) {
    const int64_t r0 = cut.start_of(w), r1 = cut.start_of(w + 1);
    if (r0 != at) ++wrong;
    at = r1;
    int64_t off = 0, t = 0;
    for (int n : len) {
      const int64_t lo = r0 > off ? r0 : off, hi = r1 < off + n ? r1 : off + n;
      off += n;
      if (lo >= hi) continue;
      if (cut.wg_of((int)lo) != w || cut.wg_of((int)hi - 1) != w) ++wrong;
      t += (hi - lo + 31) / 32;
      if (hi - lo > piece) piece = hi - lo;
    }
    if (t > tiles) tiles = t;
  }
  if (at != total) ++wrong;
  int64_t off = 0;
  for (int n : len) {
    if (n) recs += cut.wg_of((int)(off + n - 1)) - cut.wg_of((int)off) + 1;
    off += n;
  }
}

int main() {
  int S, Hkv, Hq, C, V, ld, max_L, full, L;
  while (std::scanf("%d %d %d %d %d %d %d %d %d", &S, &Hkv, &Hq, &C, &V, &ld, &max_L, &full, &L) == 9) {
    std::vector<int> len(V);
    for (int& n : len)
      if (std::scanf("%d", &n) != 1) return 1;
    if (full) len.push_back(L);
    const bd::AttnPlan f = bd::plan_attn(S, Hkv, Hq, C, V, ld, max_L, full != 0, false, true);
    const bd::AttnBwdPlan b = bd::plan_attn_bwd(S, Hkv, Hq, C, V, ld, max_L, full != 0, true);
    int64_t tiles, piece, wrong, recs, btiles, bpiece, bwrong, brecs;
    replay<bd::StreamCut<5, 4>>(len, V, f.nW, tiles, piece, wrong, recs);
    replay<bd::StreamCut<1, 1, 32>>(len, V, b.nW, btiles, bpiece, bwrong, brecs);
    const int64_t over = recs - (f.nW + f.nbr - 1);
    std::printf("%d %lld %lld %lld %d %lld %lld %lld\n", f.nW, (long long)tiles, (long long)(over > 0 ? over : 0),
                (long long)wrong, b.nW, (long long)bpiece, (long long)bwrong,
                (long long)(((int64_t)V * ld + (full ? max_L : 0) + 31) / 32));
  }
  return 0;
}
