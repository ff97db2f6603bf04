// Which way the bands of 64 rows of tall images are decoded (pilc_twar_inverse).  Host code that needs no HIP header.
//
// strips: images, or groups of whole images that share 64 rows; bands: of a strip; blocks: of 16 columns, ceil((w + 63) / 16).
//
// One at a time: a launch a band, for every strip's at once, up to four workgroups on a compute unit (k_twar_inverse_strips).
// Together: all bands of a launch follow each other (k_twar_inverse_bands), two of them on a unit or each alone on one.
//
// Whole calls, us, and what the rules below take.  (They were fitted to 10,000 random batches of up to 2048 strips, which they
// decode in 1.005 times the best of the three ways on average, one in a hundred in 1.1 times and more: rounds that are
// filled badly are guessed badly, as some rows show.)
//
//   strips x bands x columns  one   two  alone  taken
//    250 x  2 x   64     42    37    44   two
//    300 x  2 x   64     45    46    55   one
//    330 x  2 x  300     64    64    75   two
//    380 x  2 x  512     83    82    90   two
//    390 x  2 x  512     83    83   110   one
//    500 x  2 x  700     99   119   132   one
//    390 x  3 x  400    101    92   120   two
//    420 x  3 x   96     64    72    87   one
//    440 x  3 x  400    102   107   138   one
//    500 x  3 x  400    102   114   140   one
//    420 x  3 x  700    174   166   170   two
//    420 x  3 x 1500    334   337   304   one
//    420 x  5 x  256    134   128   172   two
//    500 x  5 x  256    135   146   190   one
//    420 x  8 x   96    148   149   211   one
//    380 x  8 x   96    147   136   186   two
//    420 x  8 x  256    224   203   264   two
//    500 x  4 x   64     78    87   118   one
//    760 x  4 x  400    239   237   270   one
//   1000 x  4 x  256    240   232   297   one
//   1000 x  3 x  400    250   231   268   one
//   1000 x  4 x  600    506   464   486   two
//   1500 x  8 x  150    493   537   772   one
//   1000 x  8 x  256    492   467   589   two
//    800 x  2 x 2000    572   542   528   one
//    200 x  2 x 2047    150   136   143   two
//    250 x  2 x 2047    162   184   161   one
//    256 x  3 x 2047    244   308   244   one
//    225 x  2 x 5000    338   378   378   one
//    190 x  3 x 5000    500   666   657   one
//    200 x  3 x 2047    233   238   228   alone
//    190 x  5 x 3200    554   574   511   alone
//    225 x  5 x 2047    400   486   468   one
//    200 x  4 x 2047    310   314   303   alone
//    250 x  4 x 2047    326   414   352   one
//    250 x  8 x 1300    447   529   467   one
//    190 x 12 x 1700    796   758   710   alone
//    383 x  3 x 2047    432   461   439   one
//    320 x  4 x 2047    550   492   464   alone
//    320 x  2 x 2047    265   268   222   alone
//    450 x  2 x 2047    296   340   292   one
//    256 x 17 x  900    725   817   756   one
//    240 x  4 x  945    173   177   169   one
//    256 x  3 x  945    126   121   124   two
//     30 x 17 x 1920   1095   269   215   alone
//     60 x 17 x 1920   1100   405   345   alone
//     16 x 22 x 2047   1482   251   221   alone
//     64 x 12 x   64    174    87    75   alone
//     64 x 12 x  400    284   115   100   alone
//    110 x 12 x   64    174   117    98   alone
//    120 x 12 x   64    175   111   101   two
//    112 x 12 x  400    288   134   149   two
//    145 x 12 x  100    188   143   124   alone
//    160 x 12 x  100    188   126   137   two
//    100 x  6 x   64     94    58    62   two
//     70 x  7 x  200    137    69    65   two
//    100 x  9 x  200    174    98    92   alone
//    128 x 10 x  300    213   116   124   two
//    200 x  2 x 1500    121   102   116   two
//    300 x  2 x 1000    119   103   125   two
//    180 x  3 x 1000    131   104   127   two
//    200 x  3 x 1000    132   112   128   two
//    191 x  4 x 1500    241   236   199   alone
//    128 x  4 x 1700    249   179   158   alone
//    100 x  4 x 1700    245   124   132   two
//    150 x  5 x  800    182   113   116   two
//    300 x  4 x  600    167   132   153   two
//     40 x  7 x 1000    284    99   109   two
//     50 x  7 x 1150    317   107   116   alone
#pragma once

#include <cstdint>

namespace pilc {

constexpr uint32_t kBandWords = 1u << 21;  // of a set: 8 MB, 127 bands of 16384 columns, 1057 of 1920

struct BandLaunch {  // bands together: how many of a strip and how many strips the words have room for in a launch
    uint32_t bands;
    uint64_t strips, launches;
};

static inline BandLaunch band_launches(uint64_t strips, uint32_t bands, uint32_t blocks)
{
    BandLaunch l;
    const uint64_t words = 16u * (uint64_t)blocks;  // of a band
    l.bands = bands < kBandWords / words ? bands : (uint32_t)(kBandWords / words);
    const uint64_t most = kBandWords / (l.bands * words);
    l.launches = (strips + most - 1u) / most;
    l.strips = (strips + l.launches - 1u) / l.launches;  // launches of one size
    return l;
}

// Whether the bands go one at a time.
//
// Long rows: a launch of one band of at most 256 strips, each on a unit of its own, is a round; with two, three or four on a unit
// it takes 1.75, 2.45 or 3 rounds.  Bands together, each alone on a unit, take a round for every 256 of them, and half a
// round a launch for those that get under way and those that are left over.  They have to
// be more than fit the chip two to a unit, or that is faster still.
//
// Short rows: one at a time needs strips that fill the chip by themselves, from 400 on (those that make up whole rounds do
// best), and then pays where the bands together would take long to get under way for what there is to do: two bands, or few
// blocks in all.  With two bands of less than 15 blocks it is so from one strip a unit on.
static inline bool bands_one_at_a_time(uint64_t strips, uint32_t bands, uint32_t blocks)
{
    const uint64_t on_a_unit = (strips + 255u) / 256u;
    if (blocks >= 72u || (blocks >= 60u && bands >= 4u && on_a_unit == 1u)) {
        const BandLaunch l = band_launches(strips, bands, blocks);
        if (l.launches == 1u && strips * bands <= 420u) return false;
        const uint64_t a_band = on_a_unit == 1u ? 1024u : on_a_unit == 2u ? 1792u : on_a_unit == 3u ? 2508u
                                : strips <= 1024u ? 3072u : 3u * strips;  // in 1024ths of a round
        return bands * a_band < l.launches * (4u * l.strips * bands + 512u);
    }
    if (bands == 2u && blocks <= 14u) return strips >= 256u;
    if (bands == 2u) return strips > 384u;
    const uint64_t most = strips <= 768u && strips >= 215u * on_a_unit ? 160u : 92u;
    return strips >= 400u && ((uint64_t)bands * blocks <= most || (strips >= 450u && blocks <= (strips > 1024u ? 15u : 11u)));
}

// Whether the bands of a launch have a compute unit each.  A band that has one to itself is half as fast again, and one that is
// slow holds up all below it; but two on a unit get more done.  So it pays where there are many bands that follow each
// other and units for all that are under way at the same time (a new one every thirteen blocks of a strip); and with long rows,
// where a round lasts long against the time until all bands are under way, if there are more of them than fit the chip two
// to a unit, or so many that the last ones wait for the first in any case.
static inline bool bands_alone_on_a_unit(uint64_t strips, uint32_t bands, uint32_t blocks)
{
    const uint64_t all = strips * bands;
    if (bands >= 8u && strips <= (blocks >= 9u ? 150u : 112u) && strips * (blocks + 9u) <= 3300u) return true;
    return (blocks >= 68u && (bands >= 6u || all > 560u)) || (blocks >= 110u && all > 420u);
}

}  // namespace pilc
