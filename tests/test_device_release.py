"""Where one thread writes its die's cache back to memory for blocks on other dies to read, nothing may tell them before that is done.  The
compiler drops the wait of a release fence where it knows of nothing else that is under way, so the assembly is looked at (compiled here)."""
import os
import re
import subprocess

from paper_2103_15195_amd import build as hip_build


def test_every_write_back_is_waited_for(tmp_path):
    flags = [f for f in hip_build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    names = [s for s in hip_build.SOURCES if s.startswith("kernels_")]
    jobs = [subprocess.Popen([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-S", "--cuda-device-only", *flags, "-o", str(tmp_path / (n + ".s")),
                              os.path.join(hip_build.CSRC, n)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True) for n in names]
    found = 0
    for name, job in zip(names, jobs):
        text, _ = job.communicate()
        assert job.returncode == 0, text
        kernel, code = None, []
        for line in (tmp_path / (name + ".s")).read_text().splitlines():
            line = line.split(";")[0].strip()
            label = re.match(r"(_Z\w+):$", line)
            if label:
                kernel = label.group(1)
            elif line and not line.startswith("."):
                code.append((kernel, line))
        for i, (kernel, line) in enumerate(code):
            if line.startswith("buffer_wbl2"):
                found += 1
                after = next(l for _, l in code[i + 1:] if l.startswith(("s_waitcnt", "s_endpgm", "global_", "flat_", "buffer_")))
                assert after.startswith("s_waitcnt") and "vmcnt(0)" in after, (kernel, after)
    assert found
