"""Rules that the kernels' sources keep, checked on the CPU: what they guard
against shows on the GPU only where two workgroups meet within a microsecond."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_16298_amd", "csrc")


def lines(*names):
    for name in names or sorted(os.path.basename(p) for p in glob.glob(os.path.join(CSRC, "*.h*"))):
        with open(os.path.join(CSRC, name)) as f:
            for i, line in enumerate(f, 1):
                code = line.split("//")[0]
                if code.strip():
                    yield f"{name}:{i}", code


def test_no_wave_leaves_a_pass_by_itself():
    """The passes that raise the status themselves (their bounded waits) have
    barriers: a wave that read the status and returned by itself would leave
    the others of its workgroup to go on without it."""
    alone = [(at, code.strip()) for at, code in lines("onesweep.hip", "spread.hip")
             if re.search(r"\*\s*a\.status\b.*\breturn\b", code)]
    assert alone == []


def test_no_plain_store_to_a_status_others_raise():
    """Beside workgroups that raise SS_ERR_TIMEOUT, a status computed from the
    counts is raised atomically: a load and a store could put SS_OK over a
    timeout.  The small-frame kernel alone has no waits and just stores."""
    plain = [(at, code.strip()) for at, code in lines()
             if re.search(r"\*\s*a\.status\s*=[^=]", code) and not at.startswith("tiny.hip:")]
    assert plain == []
