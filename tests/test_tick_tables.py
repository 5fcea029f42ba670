"""The tables that deal the operations of a unit to its matrix instructions are checked as they are compiled.  Here mistakes are planted in them, on the
host, and the check has to see each: an operation ahead of what it needs, one behind what needs it, an item of the other keys too early."""
import os
import shutil
import subprocess

import pytest

from paper_2505_13389_amd import build

# source -> tables with a mistake
PLANTED = {
    "fine_bwd_dkv.hip": """
struct Early : DkvTicks { constexpr Early() { ++p[PH / 2 + 2]; } };             // an exponential's argument ahead of S
struct Other : DkvTicks { constexpr Other() {                                   // of the other keys, their conversions last
  int n = 0;
  while (!(pw[n].op == CVT && pw[n].item == 7)) ++n;
  for (int t = PH / 2 + 3; t <= PH + 2; ++t) p[t] = n + 1;
} };
struct Late : DkvTicks { constexpr Late() { --p[2 * PH - 1]; } };               // P behind the first dV
struct Product : DkvTicks { constexpr Product() { ++s[2 * PH + 2]; } };         // dS ahead of dP
struct LateS : DkvTicks { constexpr LateS() { --s[3 * PH - 1]; } };             // dS behind the first dK
struct Swapped : DkvTicks { constexpr Swapped() { const Work x = pw[0]; pw[0] = pw[2]; pw[2] = x; } };  // an exponential ahead of its argument
struct Converted : DkvTicks { constexpr Converted() { const Work x = sw[1]; sw[1] = sw[3]; sw[3] = x; } };  // a conversion ahead of a product
static_assert(DkvTicks().in_order() && !Early().in_order() && !Other().in_order() && !Late().in_order() && !Product().in_order() &&
              !LateS().in_order() && !Swapped().in_order() && !Converted().in_order(), "");
static_assert(Other().pw[Other().p[DkvTicks::PH + 2] - 1].item < 8, "the last operation alone does not show it");
""",
    "fine_bwd.hip": """
struct EarlyP : DqTicks { constexpr EarlyP() { p[KS + 2] = 20; } };
struct EarlyS : DqTicks { constexpr EarlyS() { s[PH + KS + 2] = 20; } };
struct LateS : DqTicks { constexpr LateS() { s[2 * PH - 1] = 0; } };
struct Swapped : DqTicks { constexpr Swapped() { const Work x = pw[0]; pw[0] = pw[2]; pw[2] = x; } };
static_assert(DqTicks().in_order() && !EarlyP().in_order() && !EarlyS().in_order() && !LateS().in_order() && !Swapped().in_order(), "");
""",
    "fine_fwd.hip": """
template <int D> struct Early : FwdTicks<D> { constexpr Early() { ++this->ahead[this->in_pv(1)]; } };
template <int D> struct Late : FwdTicks<D> { constexpr Late() { --this->ahead[this->in_s(this->PH - 1)]; } };
template <int D> struct Swapped : FwdTicks<D> { constexpr Swapped() { const auto x = this->w[0]; this->w[0] = this->w[2]; this->w[2] = x; } };
template <int D> struct Summed : FwdTicks<D> { constexpr Summed() {  // a sum ahead of its exponential
  int n = 0;
  while (this->w[n].op != this->ADD) ++n;
  const auto x = this->w[n]; this->w[n] = this->w[2]; this->w[2] = x;
} };
template <int D> constexpr bool seen = FwdTicks<D>().in_order() && !Early<D>().in_order() && !Late<D>().in_order() && !Swapped<D>().in_order() && !Summed<D>().in_order();
static_assert(seen<128> && seen<64>, "");
""",
}


@pytest.mark.parametrize("source", PLANTED)
def test_a_planted_mistake_is_seen(source, tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("no compiler")
    unit = tmp_path / source
    unit.write_text(f'#include "{os.path.join(build.CSRC, source)}"\nnamespace vsa {{{PLANTED[source]}}}\n')
    r = subprocess.run(["hipcc", *build.FLAGS, f"-I{build.CSRC}", "-fsyntax-only", str(unit)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
