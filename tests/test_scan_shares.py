"""Which pairs of words a wave looks at in the completion pass where steps overlap (host code of the step kernel's header, on the CPU): every
pair has one wave whatever number of waves serve, and no wave has more than one round of them, up to the most words of either
size of workgroup."""
import os
import subprocess
import textwrap

from paper_2602_02987_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_pair_of_words_has_one_wave(tmp_path):
    src = tmp_path / "shares.hip"
    src.write_text(textwrap.dedent("""
        #include <cstdio>
        #include "gnr_step.h"
        using namespace gnr;
        int main()
        {
          struct { int nwaves; bool beside; int words; } forms[] = {
              {8, false, kMostWordsEight}, {8, true, kMostWordsEight}, {16, true, kStaticWordsMedium}, {16, true, kStaticWordsLarge}};
          long looked = 0;
          for (auto f : forms)
            for (int words = 1; words <= f.words; ++words) {
              const int npairs = (words + 1) / 2, drain = event_waves(f.nwaves, f.beside, words);
              if (drain < 1 || drain > f.nwaves) { std::printf("%d waves, %d words: %d\\n", f.nwaves, words, drain); return 1; }
              for (int serve = 1; serve <= f.nwaves; ++serve) {
                int owners[kStaticWordsLarge] = {};
                for (int wave = f.nwaves - drain; wave < f.nwaves; ++wave) {
                  const Scan s = scan_of(wave, f.nwaves, words, drain, serve, f.beside);
                  int mine = 0;
                  for (int p = s.first; p < s.end; p += s.stride, ++mine) ++owners[p];
                  if (mine > kPairsARound || s.end > npairs) { std::printf("%d waves, %d words, %d serve: %d pairs\\n", f.nwaves, words, serve, mine); return 1; }
                }
                for (int p = 0; p < npairs; ++p, ++looked)
                  if (owners[p] != 1) { std::printf("%d waves, %d words, %d serve: pair %d has %d\\n", f.nwaves, words, serve, p, owners[p]); return 1; }
                // the kernel divides by a reciprocal, which may be off by an ulp
                const int busy = serve < drain ? serve : drain, share = 2 * (drain - busy) + busy;
                for (float off : {-1.2e-7f, 0.0f, 1.2e-7f}) {
                  const int each = static_cast<int>((static_cast<float>(npairs + share) - 0.5f) * (1.0f / share * (1.0f + off)));
                  if (each != (npairs + share - 1) / share) { std::printf("%d pairs, %d shares: %d\\n", npairs, share, each); return 1; }
                }
              }
            }
          if (a_round_is_enough(8, true, kStaticWordsLarge)) { std::printf("the bound bounds nothing\\n"); return 1; }
          std::printf("clean %ld\\n", looked);
          return 0;
        }
        """))
    exe = str(tmp_path / "shares")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-Xclang", "-target-feature", "-Xclang",
                           "-packed-fp32-ops", f"-I{os.path.join(ROOT, 'include')}", f"-I{os.path.join(ROOT, 'paper_2602_02987_amd', 'csrc')}",
                           str(src), "-o", exe], stderr=subprocess.DEVNULL)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and res.stdout.startswith("clean"), (res.stdout, res.stderr)


def test_more_words_take_sixteen_waves():
    """What the bound of eight waves rests on: configurations beyond 5120 servers are never given fewer than sixteen."""
    from paper_2602_02987_amd import binding as B
    for N in (5119, 5120, 5121, 5184, 6000, 8191, 10_240, 11_000):
        for route in (W.ROUTE_SOLO_FIRST, W.ROUTE_RANDOM_SPLIT, W.ROUTE_IMMEDIATE, W.ROUTE_WEIGHTED_SPLIT):
            for theta in (0.0, 0.1):
                cls = [W.SimClass(lam=0.01, in_p0=100.0, out_p0=50.0, theta=theta) for _ in range(2)]
                cfg = W.SimConfig(name="words", K=2, N=N, B=8, C=256, c0=0.01, c_pre=0.0, c_dec=0.0, classes=cls, M=0, x_star=[0.1] * 2,
                                  qp_star=[0.0] * 2, route_mode=route, p_solo=[0.5] * 2, w_solo=[0.5] * 2, w_mixed=[0.5] * 2)
                for replications in (1, 300, 700, 3000):
                    threads = B.sim_launch_plan(cfg, replications)[0]
                    assert N <= 5120 or threads == 1024
