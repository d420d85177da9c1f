"""The counted traffic that bench.py reports belongs to one state of a kernel: it is dropped as soon as any
file that the kernel is built from changes, its headers among them."""
import hashlib
import os
import shutil

import bench


def test_counted_traffic_is_dropped_when_a_source_changes(tmp_path, monkeypatch):
    for kernel, entry in bench.MEASURED_TRAFFIC.items():
        csrc = os.path.join(bench.ROOT, bench.CSRC)
        used, sha = set(entry["sources"]), hashlib.sha1()
        for name in entry["sources"]:
            with open(os.path.join(csrc, name)) as f:
                text = f.read()
            sha.update(text.encode())
            used.update(l.split('"')[1] for l in text.splitlines() if l.startswith('#include "'))
        # (the header of plain declarations changes with every kernel of the library)
        assert used - {"dynb_internal.h"} == set(entry["sources"]), kernel
        for changed in entry["sources"]:
            root = tmp_path / kernel / changed
            (root / bench.CSRC).mkdir(parents=True)
            for name in entry["sources"]:
                shutil.copy(os.path.join(csrc, name), root / bench.CSRC / name)
            with monkeypatch.context() as m:
                m.setitem(bench.MEASURED_TRAFFIC, kernel, dict(entry, sha1=sha.hexdigest()[:12]))
                m.setattr(bench, "ROOT", str(root))
                assert bench.measured_traffic(kernel, 4) == entry["bytes_per_launch"]
                assert bench.measured_traffic(kernel, 3) is None
                with open(root / bench.CSRC / changed, "a") as f:
                    f.write("\n")
                assert bench.measured_traffic(kernel, 4) is None, changed
