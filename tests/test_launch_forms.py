"""What the launch rule promises, whatever shapes it takes (host code, on the CPU; the step kernel's variants are stubs that note which
form they are asked for): sizes that exist and fit, no allowed workgroup with fewer rounds, rounds with few waves counting
more, the dense form where it saves a round, and the form reported is the one that a launch asks for."""
import os
import subprocess
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launch_rule_and_the_forms_it_leads_to(tmp_path):
    src = tmp_path / "forms.hip"
    src.write_text(textwrap.dedent("""
        #include <cstdio>
        #include <cstring>
        #include <random>
        #include "gnr_step.h"
        namespace gnr {
        static int asked_variant, asked_form; static bool asked_dense;
        static StepKernel note(int variant, int form, bool dense) { asked_variant = variant; asked_form = form; asked_dense = dense; return nullptr; }
        StepKernel step_kernel_plain(int f, bool d) { return note(0, f, d); }
        StepKernel step_kernel_rr(int f, bool d) { return note(1, f, d); }
        StepKernel step_kernel_im(int f, bool d) { return note(2, f, d); }
        StepKernel step_kernel_ab(int f, bool d) { return note(3, f, d); }
        StepKernel step_kernel_ab_rr(int f, bool d) { return note(4, f, d); }
        StepKernel step_kernel_ab_im(int f, bool d) { return note(5, f, d); }
        StepKernel step_kernel_ws(int f, bool d) { return note(6, f, d); }
        }
        using namespace gnr;
        static const int kCompiledFor[7] = {64, 128, 256, 512, 1024, 1024, 512};
        // rounds of a launch on 256 compute units with 160 KB and four SIMDs of `per_simd` waves each; a round with w waves on a compute
        // unit, fewer than eight, counts as 8 / w of one (in 840ths)
        static long rounds_of(int reps, int threads, size_t lds, int per_simd, long *weighed)
        {
          const long by_waves = 4l * per_simd / (threads / 64), by_lds = static_cast<long>(163840 / lds);
          long wgs = by_waves < by_lds ? by_waves : by_lds;
          if (wgs < 1) wgs = 1;
          const long rounds = (reps + 256 * wgs - 1) / (256 * wgs), waves = wgs * threads / 64;
          if (weighed) *weighed = rounds * (840 / (waves < 8 ? waves : 8));
          return rounds;
        }
        int main()
        {
          std::mt19937 rng(20);
          auto upto = [&](int n) { return static_cast<int>(rng() % static_cast<unsigned>(n)); };
          long tried = 0;
          for (int it = 0; it < 60000; ++it) {
            Params q;
            std::memset(&q, 0, sizeof q);
            q.K = 1 + upto(kMaxK);
            q.N = it % 3 ? 1 + upto(1 << (1 + upto(13))) : 1 + upto(11500);
            q.route_mode = SIM_ROUTE_SOLO_FIRST;
            for (int mode : {SIM_ROUTE_SOLO_FIRST, SIM_ROUTE_RANDOM_SPLIT, SIM_ROUTE_IMMEDIATE, SIM_ROUTE_WEIGHTED_SPLIT})
              if (upto(4) == 0) q.route_mode = mode;
            q.Mp = q.M = q.route_mode == SIM_ROUTE_IMMEDIATE ? q.N : upto(q.N + 1);
            q.nwords = (q.N + 63) / 64;
            q.tbt_w = 1 + upto(90);
            if (upto(2)) q.ab_classes = 1;
            q.dl_rings = q.ab_classes != 0 || q.route_mode == SIM_ROUTE_WEIGHTED_SPLIT;
            const int reps = 1 + upto(1 << (1 + upto(13)));
            const int threads = step_threads(q, reps);
            q.threads = threads;
            const size_t lds = step_lds_bytes(q);
            const bool dense = step_dense(reps, threads, lds);
        #define FAIL(what) { std::printf("%s: K %d N %d M %d route %d rings %d reps %d: %d threads, %zu bytes\\n", what, q.K, q.N, q.M, q.route_mode, q.dl_rings, reps, threads, lds); return 1; }
            if (threads < 64 || threads > 1024 || (threads & (threads - 1))) FAIL("no such size");
            if (q.N > 64 * kMostWordsEight && threads != 1024) FAIL("few waves for many words");
            if (lds > 163840) continue;   // (refused by the configuration checks)
            ++tried;
            long mine, other;
            const long rounds4 = rounds_of(reps, threads, lds, 4, &mine), rounds2 = rounds_of(reps, threads, lds, 2, nullptr);
            if (dense != (threads <= 512 && rounds4 < rounds2)) FAIL("dense form");
            if (q.N <= 64 * kMostWordsEight)
              for (int t = 64; t <= threads; t *= 2) {   // no smaller one would need less (larger ones have their own limits)
                Params o = q;
                o.threads = t;
                const size_t bytes = step_lds_bytes(o);
                rounds_of(reps, t, bytes, 4, &other);
                if (other < mine) FAIL("a smaller workgroup needs fewer rounds");
              }
            asked_form = -1;
            const int rc = launch_steps(q, reps, threads, lds, 0, 1, nullptr);   // (the stubs have no kernel: refused before any launch)
            const bool two = q.route_mode == SIM_ROUTE_RANDOM_SPLIT;
            const int variant = q.route_mode == SIM_ROUTE_WEIGHTED_SPLIT ? 6 : (q.dl_rings ? 3 : 0) + (two ? 1 : q.route_mode == SIM_ROUTE_IMMEDIATE ? 2 : 0);
            if (rc != SIM_EINVAL || asked_form < 0 || asked_form > 6 || asked_variant != variant) FAIL("variant");
            if (kCompiledFor[asked_form] != threads || asked_dense != dense) FAIL("form launched");
            if (threads == 1024 && static_words(asked_form - 2) < q.nwords) FAIL("layout");
          }
          std::printf("clean %ld\\n", tried);
          return tried < 40000;
        }
        """))
    exe = str(tmp_path / "forms")
    csrc = os.path.join(ROOT, "paper_2602_02987_amd", "csrc")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                           f"-I{os.path.join(ROOT, 'include')}", f"-I{csrc}", str(src), os.path.join(csrc, "gnr_kernels.hip"), "-o", exe],
                          stderr=subprocess.DEVNULL)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.startswith("clean"), (res.stdout, res.stderr)
