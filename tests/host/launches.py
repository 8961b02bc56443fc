"""Calls made of the library beside a stand-in for the launch (launch_recorder.cpp): what each would launch, as JSON.

argv: the stand-in, the library, a JSON list of calls [dims, layout, cb, wt_is_packed] of conv2d_int8_ex, or with a tile and a depth split
behind that, of conv2d_int8_packed, or with "requant" in the place of wt_is_packed and out_cb, out_pad behind it, of conv2d_int8_packed_requant.  The stand-in is loaded first, so the
library's launches go to it; no memory is touched.
"""
import ctypes
import json
import sys

recorder = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
recorded, name = (ctypes.c_int * 4).in_dll(recorder, "recorded"), (ctypes.c_char * 512).in_dll(recorder, "recorded_name")
p, big = ctypes.c_void_p(1 << 20), ctypes.c_size_t(1 << 40)
out = []
for dims, layout, cb, packed, *forced in json.loads(sys.argv[3]):
    d = (ctypes.c_int * 9)(*dims)
    before = recorded[0]
    if packed == "requant":
        rc = lib.conv2d_int8_packed_requant(d, layout, cb, p, p, p, *forced, 9, 1, None)
        out.append(dict(rc=rc, launches=recorded[0] - before, workgroups=recorded[1], kernel=name.value.decode()))
        continue
    rc = lib.conv2d_int8_packed(d, layout, cb, p, p, p, *forced, None) if forced else lib.conv2d_int8_ex(d, layout, cb, p, p, packed, p, p, big, None)
    v = [ctypes.c_int() for _ in range(3)]
    lib.conv2d_int8_query_stage(d, 1, layout, cb, packed, 1, *map(ctypes.byref, v))
    out.append(dict(rc=rc, launches=recorded[0] - before, workgroups=recorded[1], threads=recorded[2], lds=recorded[3], kernel=name.value.decode(), stage=[x.value for x in v]))
print(json.dumps(out))
