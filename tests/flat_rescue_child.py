"""Child process of the flat look-back's rescue test (run with SKEL_LIBRARY naming
the library whose flat tiles wait for one poll only): scans and row scans whose
tiles compute most of their predecessors' totals themselves, against torch, with
the same bits on every repeat."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import torch  # noqa: E402

import paper_1405_2915_amd as skel  # noqa: E402

TYPES = {skel.F32: torch.float32, skel.I32: torch.int32, skel.I64: torch.int64}


def check(name, call, rows, cols, din, dout, kind):
    dev = "cuda"
    x = (torch.randn(rows, cols, device=dev) if din == skel.F32 else
         torch.randint(-1000, 1000, (rows, cols), device=dev, dtype=TYPES[din]))
    v = x.flip(1) if kind >= 2 else x
    ref = v.to(torch.float64 if din == skel.F32 else torch.int64).cumsum(1)
    mag = v.abs().double().cumsum(1)
    if kind % 2:
        ref = ref - v
    ref, mag = (ref.flip(1), mag.flip(1)) if kind >= 2 else (ref, mag)
    y = torch.empty(rows, cols, device=dev, dtype=TYPES[dout])
    cx, cy = skel.wrap_tensor(x), skel.wrap_tensor(y)
    first = None
    print(name, rows, cols, din, dout, kind, flush=True)
    for rep in range(5):
        y.fill_(-1)
        call(cx, cy, kind)
        if din == skel.F32:
            assert bool(((y - ref).abs() <= 1e-5 * mag).all()), rep
        else:
            assert torch.equal(y, ref.to(TYPES[dout])), rep
        first = y.clone() if first is None else first
        assert torch.equal(y, first), rep
    skel.skel_sync()
    cx.destroy()
    cy.destroy()


def main():
    assert skel.LIB_PATH == os.environ.get("SKEL_LIBRARY"), "not the stress build"
    skel.skel_init(0, "torch")
    pairs = [(skel.F32, skel.F32), (skel.I32, skel.I32), (skel.I32, skel.I64),
             (skel.I64, skel.I64)]
    for din, dout in pairs:
        for kind in range(4):
            scan = lambda v: lambda a, b, k: skel.skel_scan(a, b, k, skel.SUM,  # noqa: E731
                                                            variant=v)
            check("S5", scan(5), 1, 300003, din, dout, kind)
            check("S3", scan(3), 1, 2000003, din, dout, kind)
            rows = lambda a, b, k: skel.skel_scan_rows(a, b, k, skel.SUM,  # noqa: E731
                                                       variant=1)
            check("SR1", rows, 1, 500001, din, dout, kind)
            check("SR1", rows, 9, 60007, din, dout, kind)
    print("ok", flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
