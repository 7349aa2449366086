"""Which kernels a call of the library launches, without a GPU.

record(calls) runs the calls in a process of its own, where launch_recorder.c
takes the place of the HIP launch calls, and returns for each the list of its
launches [(mangled kernel name, grid x, grid y, grid z)] (for "ws" the size).
The pointers are never read: the entry points only check them.
A call is a dict: "dims" (T, d, n, E, K) and "call", one of
  route  moe_route with "flags"
  fwd    moe_fwd on the routing of route, or with "round" = (m_tile, mode) of moe_round_tokens
  bwd    moe_bwd on the same; "dbias", "dS": whether they are asked for
  ws     moe_workspace_bytes of "which", with the default or given "capacity"
and "cus", the CUs that the device reports (256; the library asks once per process).
"""
import ctypes
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))


def record(calls, tmp_path):
    so = os.path.join(str(tmp_path), "launch_recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_recorder.c")], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), so], input=json.dumps(calls), text=True,
                       capture_output=True, cwd=os.path.dirname(HERE))
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout)


def _routing(B, D, capacity):
    r = B.MoeRouting()
    r.capacity, r.words = capacity, (D.T + 63) // 64
    for i, name in enumerate(B.MoeRouting.pointer_fields()):
        setattr(r, name, 0x10000000 + 0x1000 * i)
    return r


def _main():
    rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    rec.rec_name.restype = ctypes.c_char_p
    sys.path.insert(0, os.path.dirname(HERE))
    from paper_2512_14080_amd import binding as B
    L = B.lib()
    out = []
    p, ws = 0x20000000, (0x30000000, 1 << 62)

    def ok(rc):
        assert rc == B.MOE_OK, B.moe_last_error()

    for c in json.load(sys.stdin):
        D = B.dims(*c["dims"])
        rec.rec_set_cus(c.get("cus", 256))
        cap = c.get("capacity", D.T * D.K)
        if c["call"] == "ws":
            out.append(B.moe_workspace_bytes(D, cap, c["which"]))
            continue
        rec.rec_clear()
        r = _routing(B, D, cap)
        ok(L.moe_route(D, p, p, None, c.get("flags", 0), ctypes.byref(r), None))
        if c["call"] != "route":
            if "round" in c:
                tc, r = r, _routing(B, D, B.moe_round_capacity(D, c["round"][0]))
                r.mask = tc.mask + 64
                ok(L.moe_round_tokens(D, c["round"][0], B.ROUND_MODES[c["round"][1]], p, ctypes.byref(tc),
                                      ctypes.byref(r), None))
            rec.rec_clear()
            if c["call"] == "fwd":
                ok(L.moe_fwd(D, p, p, p, None, ctypes.byref(r), p, p, *ws, None))
            else:
                ok(L.moe_bwd(D, p, p, p, p, p, None, p, ctypes.byref(r), p, p, p, p, p if c["dbias"] else None,
                             p if c.get("dS") else None, *ws, None))
        out.append([(rec.rec_name(i).decode(), *(rec.rec_grid(i, a) for a in range(3))) for i in range(rec.rec_count())])
    print(json.dumps(out))


if __name__ == "__main__":
    _main()
