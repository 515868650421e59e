// Instantiations and launcher of the grouped (mixture-of-experts) form of the one-shot decode kernels
// (tm_w4_stream_impl.h), 4-bit weights, experts with up to eight or sixteen rows per pass.
#include "tm_w4_stream_impl.h"

namespace tmw4 {

namespace {

template <int NTW, int NI>
hipError_t launch_grouped_ni(const GroupedParams& gp, int experts, int group, int block, hipStream_t stream)
{
    return block > 512   ? launch_stream_grouped_cfg<NTW, NI, 16>(gp, experts, group, block, stream)
           : block > 256 ? launch_stream_grouped_cfg<NTW, NI, 8>(gp, experts, group, block, stream)
                         : launch_stream_grouped_cfg<NTW, NI, 4>(gp, experts, group, block, stream);
}

template <int NTW>
hipError_t launch_grouped_ntw(const GroupedParams& gp, int experts, int group, int ni, int block, hipStream_t stream)
{
    switch (ni) {
        case 1: return launch_grouped_ni<NTW, 1>(gp, experts, group, block, stream);
        case 2: return launch_grouped_ni<NTW, 2>(gp, experts, group, block, stream);
        case 3: return launch_grouped_ni<NTW, 3>(gp, experts, group, block, stream);
        case 4: return launch_grouped_ni<NTW, 4>(gp, experts, group, block, stream);
        case 6: return launch_grouped_ni<NTW, 6>(gp, experts, group, block, stream);
        case 8: return launch_grouped_ni<NTW, 8>(gp, experts, group, block, stream);
        default: return hipErrorInvalidValue;
    }
}

template <int NTW, int NI>
hipError_t raise_grouped_ntw_ni()
{
    hipError_t e = hipSuccess;
    auto acc = [&](hipError_t r) { if (e == hipSuccess) e = r; };
    acc(stream_grouped_raise_one<NTW, 1, NI, 16>());
    acc(stream_grouped_raise_one<NTW, 2, NI, 16>());
    acc(stream_grouped_raise_one<NTW, 4, NI, 16>());
    acc(stream_grouped_raise_one<NTW, 1, NI, 8>());
    acc(stream_grouped_raise_one<NTW, 1, NI, 4>());
    acc(stream_grouped_raise_one<NTW, 2, NI, 8>());
    acc(stream_grouped_raise_one<NTW, 2, NI, 4>());
    acc(stream_grouped_raise_one<NTW, 4, NI, 8>());
    acc(stream_grouped_raise_one<NTW, 4, NI, 4>());
    return e;
}

template <int NTW>
hipError_t raise_grouped_ntw()
{
    hipError_t e = raise_grouped_ntw_ni<NTW, 1>();
    if (e == hipSuccess) e = raise_grouped_ntw_ni<NTW, 2>();
    if (e == hipSuccess) e = raise_grouped_ntw_ni<NTW, 3>();
    if (e == hipSuccess) e = raise_grouped_ntw_ni<NTW, 4>();
    if (e == hipSuccess) e = raise_grouped_ntw_ni<NTW, 6>();
    if (e == hipSuccess) e = raise_grouped_ntw_ni<NTW, 8>();
    return e;
}

}  // namespace

hipError_t stream_grouped_setup()
{
    hipError_t e = raise_grouped_ntw<1>();
    if (e == hipSuccess) e = raise_grouped_ntw<2>();
    if (e == hipSuccess) e = raise_grouped_ntw<3>();
    if (e == hipSuccess) e = raise_grouped_ntw<4>();
    if (e == hipSuccess) e = raise_grouped_ntw<5>();
    if (e == hipSuccess) e = raise_grouped_ntw<6>();
    if (e == hipSuccess) e = raise_grouped_ntw<7>();
    if (e == hipSuccess) e = raise_grouped_ntw<8>();
    return e;
}

// Small CTAs for experts with few rows, where the K range allows: sixteen waves per CU in CTAs of four waves (K up to 2048) or
// eight (up to 4096).  `rows`: rows of an expert to size for; active: experts that can have rows.  A wave takes a quarter (an
// eighth) of the K units and as many column tiles as keep its weights in flight to 64 registers - with four waves 48: two tiles
// of four units ran 20 % faster than three - and the launch at two CTAs per CU.  LDS is sized for sixteen rows where sixteen waves'
// share allows it, else for eight (an expert with more takes a second pass), else the form is not taken.  Eight waves with groups of
// 64 do not pay: 128 experts of 4096 x 3072, 16 / 64 tokens x 8: 120 / 183 us, 109 / 160 on the large CTAs (groups of 128: 104 / 157
// and 124 / 170; of 32: 132 / 205 and 162 / 229).
bool stream_grouped_form(int NT, int KU, int group, int active, double rows, int num_cu, Plan* one, int* pass_log, int* lds)
{
    const int gpu = 128 / group;
    const int waves = KU <= 16 ? 4 : 8;
    const int need = (KU + waves - 1) / waves;
    if (need > 4) return false;
    const int ni = need;                                   // 1 ... 4: all built
    int ntw = (waves == 4 ? 48 : 64) / (ni * (4 + gpu));
    ntw = ntw > 4 ? 4 : ntw;
    if (waves == 4 && ntw > 3) ntw = 3;
    while (ntw > 1 && (long)active * ((NT + ntw - 1) / ntw) < 2 * num_cu) --ntw;
    if (ntw < 1 || !grouped_small_built(ntw, gpu, ni, waves)) return false;
    const size_t share = 160 * 1024 / (16 / waves) - 512;  // of the CU's LDS, for one of the resident CTAs
    for (int log = 4; log >= 3; --log) {
        int red_off;
        const size_t bytes = stream_lds_bytes(ni, log, ntw, waves, share, &red_off);
        if (bytes > share) continue;
        if (rows > (1 << log)) return false;
        *one = Plan{};
        one->strips = (NT + ntw - 1) / ntw;
        one->split = 1;
        one->stream_ni = ni;
        one->block = (unsigned)waves * 64;
        *pass_log = log;
        *lds = (int)bytes;
        return true;
    }
    return false;
}

// ni units per wave and block threads, gp.pass_rows and gp.lds_bytes as the dispatcher chose them.
hipError_t launch_stream_grouped(const GroupedParams& gp, int experts, int group, int ni, int block, hipStream_t stream)
{
    if (experts <= 0 || experts > 65535 || gp.strips <= 0 || (size_t)gp.lds_bytes > kStreamLdsBudget) return hipErrorInvalidValue;
    const int ntw = gp.strip_base + (gp.strip_rem > 0 ? 1 : 0);
    switch (ntw) {
        case 1: return launch_grouped_ntw<1>(gp, experts, group, ni, block, stream);
        case 2: return launch_grouped_ntw<2>(gp, experts, group, ni, block, stream);
        case 3: return launch_grouped_ntw<3>(gp, experts, group, ni, block, stream);
        case 4: return launch_grouped_ntw<4>(gp, experts, group, ni, block, stream);
        case 5: return launch_grouped_ntw<5>(gp, experts, group, ni, block, stream);
        case 6: return launch_grouped_ntw<6>(gp, experts, group, ni, block, stream);
        case 7: return launch_grouped_ntw<7>(gp, experts, group, ni, block, stream);
        case 8: return launch_grouped_ntw<8>(gp, experts, group, ni, block, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tmw4
