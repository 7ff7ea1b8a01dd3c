"""The bench names the launch that the library makes: its chunk-count limits are
the ones in the library's sources."""
import os
import re

import bench
import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _limit(name, file="internal.hpp"):
    with open(os.path.join(ROOT, "paper_2307_03760_amd", "csrc", file)) as f:
        return int(re.search(rf"\b{name} = (\d+)", f.read()).group(1))


def test_descriptions_change_at_the_limits():
    for codec, name, file, below, above in [
            (oracle.RLE_V1, "kSplitMaxChunks", "internal.hpp", "rle_v1_index", "decode_plain"),
            (oracle.RLE_V2, "kV2BlocksMaxChunks", "internal.hpp", "rle_v2_blocks", "rle_v2_index"),
            (oracle.RLE_V2, "kSplitV2MaxChunks", "internal.hpp", "rle_v2_index", "decode_plain"),
            (oracle.DEFLATE, "kBigTeamMaxChunks", "team.hip", "16 waves", "8 waves"),
            (oracle.DEFLATE, "kTeamMaxChunks", "internal.hpp", "deflate_team", "decode_plain<DEFLATE>"),
            (oracle.LZ4, "kLzGrid", "team.hip", "a workgroup of 16", "256 workgroups"),
            (oracle.LZ4, "kLzTeamMaxChunks", "internal.hpp", "lz4_team", "decode_plain<LZ4>"),
            (oracle.BYTE_RLE, "kByteBlocksMaxChunks", "internal.hpp", "byte_rle_blocks", "decode_plain")]:
        n = _limit(name, file)
        assert below in bench.launch_description(codec, n), (codec, n)
        assert above in bench.launch_description(codec, n + 1), (codec, n + 1)
        assert below in bench.launch_description(codec, 1) or codec == oracle.RLE_V2
