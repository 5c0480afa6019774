"""The counter summaries see every kernel that attends or merges, each under its own name."""
import csv
import glob
import os
import re
import sys

from bench_support import pmc_summary

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def kernels():
    src = "".join(open(p).read() for p in sorted(glob.glob(
        os.path.join(ROOT, "paper_2411_01783_amd", "csrc", "*.h*"))))
    names = re.findall(r"__global__[^(]*\([^)]*\)[^(]*?(\w+_kernel)\(", src)
    return [n for n in names if re.search("prefill|decode|merge", n)]


def test_every_kernel_has_a_summary_of_its_own(tmp_path, monkeypatch):
    names = kernels()
    assert len(names) >= 9 and len(set(names)) == len(names)

    def write(path, counter):
        with open(path, "w", newline="") as f:
            out = csv.writer(f)
            out.writerow(["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"])
            out.writerow([0, "void at::native::MulFunctor<float>", counter, 1 << 18])
            for i, n in enumerate(names):
                out.writerow([i + 1, "void cp::(anonymous namespace)::%s<float, 4>(cp::X)" % n,
                              counter, 100 + i])
    fetch, wrote = str(tmp_path / "f.csv"), str(tmp_path / "w.csv")
    write(fetch, "FETCH_SIZE")
    write(wrote, "WRITE_SIZE")
    monkeypatch.setattr(sys, "argv", ["pmc_summary", fetch, wrote, str(tmp_path), "prefill_128k", "cmd"])
    pmc_summary.main()
    files = glob.glob(str(tmp_path / "*_hbm_traffic.txt"))
    assert len(files) == len(names)
    for path in files:
        assert "dispatches: 1\n" in open(path).read()
        assert os.path.basename(path).startswith("decode") == path.endswith("decode_b32_hbm_traffic.txt")
