"""Which kernels a call would launch (host side, no GPU needed)."""
import ctypes

import paper_2502_04507_amd as sta


def launches(B, H, D, grid, tile, windows, gradients=False, workspace=False):
    """The lines of sta_describe_launches; windows: one for all heads or one per head."""
    per_head = [windows[h % len(windows)] for h in range(H)]
    flat = (ctypes.c_int * (3 * H))(*[x for w in per_head for x in w])
    text = ctypes.create_string_buffer(1 << 14)
    I3 = ctypes.c_int * 3
    status = sta.load_library().sta_describe_launches(int(gradients), B, H, D, I3(*grid), I3(*tile), flat, int(workspace), text,
                                                      ctypes.c_size_t(len(text)))
    assert status == 0, sta.sta_strerror(status)
    return text.value.decode().splitlines()
