"""The traffic records' digest covers every file with device code that the
measured kernels are built from."""
import re

from paper_1710_07041_amd import traffic


def included(rel, seen):
    """The csrc files that rel includes, transitively, itself among them."""
    if rel in seen:
        return
    seen.add(rel)
    for name in re.findall(r'#include "([^"]+)"', (traffic.PKG / rel).read_text()):
        if (traffic.PKG / "csrc" / name).exists():
            included("csrc/" + name, seen)


def test_digest_covers_device_code():
    seen = set()
    for rel in traffic.KERNEL_SOURCES:
        included(rel, seen)
    device = {rel for rel in seen if "__device__" in traffic._code_only((traffic.PKG / rel).read_text())}
    assert device <= set(traffic.KERNEL_SOURCES)
