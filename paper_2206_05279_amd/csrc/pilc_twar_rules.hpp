// Which way the bands of 64 rows of tall images are decoded (pilc_twar_inverse).  Host code that needs no HIP header.
//
// strips: images, or groups of whole images that share 64 rows; bands: of a strip; blocks: of 16 columns, ceil((w + 63) / 16).
//
// One at a time: a launch a band, for every strip's at once, up to four workgroups on a compute unit (k_twar_inverse_strips).
// Together: all bands of a launch follow each other (k_twar_inverse_bands), two of them on a unit or each alone on one.
//
// Whole calls, us, and what the rules below take.  (They were fitted to 40,000 random batches of 16 to 2048 strips, which they
// decode in 1.003 times the best of the three ways on average, one in two hundred in 1.1 times and more.)
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
//    440 x  3 x  400    102   107   138   two
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
//   1000 x  3 x  400    250   231   268   two
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
//    120 x 12 x   64    175   111   101   alone
//    112 x 12 x  400    288   134   149   two
//    145 x 12 x  100    188   143   124   alone
//    160 x 12 x  100    188   126   137   two
//    100 x  6 x   64     94    58    62   two
//     70 x  7 x  200    137    69    65   alone
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
//     442 x  4 x  253    115   120   146   one
//     438 x  5 x   69     99   102   136   one
//     460 x  6 x  264    173   173   219   one
//     465 x 10 x  159    223   237   328   one
//     500 x  4 x  711    267   270   270   one
//     493 x  9 x  229    237   262   340   one
//     509 x 17 x  165    374   418   576   one
//     553 x  5 x  252    179   170   218   two
//     535 x  8 x   53    163   171   237   one
//     684 x  9 x  158    260   296   408   one
//     681 x  9 x  274    388   412   497   two
//     795 x  4 x  269    204   186   243   two
//     861 x  9 x   96    302   327   457   one
//    1011 x 10 x  130    441   452   618   one
//    1064 x  8 x  198    428   431   569   one
//    1045 x  8 x  260    501   489   614   two
//    1409 x  5 x  244    390   415   534   one
//     212 x  2 x 1101    102    80    98   two
//     303 x  2 x 1305    168   148   155   two
//     534 x  2 x  972    222   200   206   two
//     814 x  2 x  916    297   262   278   two
//      49 x 10 x  854    366   133   112   alone
//     135 x  9 x  737    306   198   194   alone
//     100 x  7 x  122    125    80    71   alone
//     114 x 12 x   54    175   117    98   alone
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
// Short rows, and two bands of any but the longest: one at a time needs strips that fill the chip by themselves, from 385 on, and
// pays by how well they make up whole rounds (with two on a unit from 471 strips on always; a third of a round
// left empty is more than together ever loses), and then where the bands together would take long to get
// under way for what there is to do: few blocks, or few in all.  With two bands of less than 15 blocks it is so from
// one strip a unit on.
static inline bool bands_one_at_a_time(uint64_t strips, uint32_t bands, uint32_t blocks)
{
    const uint64_t on_a_unit = (strips + 255u) / 256u;
    if (bands == 2u && blocks < 110u) {
        if (blocks <= 14u) return strips >= 256u;
        const bool little_over = (strips > 512u && strips <= 600u) || (strips > 768u && strips <= 900u && blocks < 75u);
        return strips > 384u && !(blocks >= 45u && little_over);
    }
    if (blocks >= 72u || (blocks >= 60u && bands >= 4u && on_a_unit == 1u)) {
        const BandLaunch l = band_launches(strips, bands, blocks);
        if (l.launches == 1u && strips * bands <= 420u) return false;
        const uint64_t a_band = on_a_unit == 1u ? 1024u : on_a_unit == 2u ? 1792u : on_a_unit == 3u ? 2508u
                                : strips <= 1024u ? 3072u : 3u * strips;  // in 1024ths of a round
        return bands * a_band < l.launches * (4u * l.strips * bands + 512u);
    }
    if (strips >= 471u && strips <= 512u) return true;
    // up to so many blocks of a row, or so many of a strip
    const struct {
        uint32_t from, row, strip;
    } lines[] = {{1281u, 23u, 80u}, {1025u, 19u, 80u}, {942u, 15u, 80u}, {820u, 11u, 80u}, {769u, 0u, 80u}, {707u, 26u, 224u},
                 {615u, 17u, 112u}, {513u, 11u, 80u},  {451u, 19u, 136u}, {411u, 7u, 80u}};
    for (const auto &l : lines)
        if (strips >= l.from) return blocks <= l.row || (uint64_t)bands * blocks <= l.strip;
    return false;
}

// Whether the bands of a launch have a compute unit each.  A band that has one to itself is half as fast again, and one that is
// slow holds up all below it; but two on a unit get more done.  So it pays where there are many bands that follow each
// other and units for all that are under way at the same time (a new one every thirteen blocks of a strip); and with long rows,
// where a round lasts long against the time until all bands are under way, if there are more of them than fit the chip two
// to a unit, or so many that the last ones wait for the first in any case.
static inline bool bands_alone_on_a_unit(uint64_t strips, uint32_t bands, uint32_t blocks)
{
    const uint64_t all = strips * bands;
    if (bands >= 8u && strips <= (blocks >= 9u ? 150u : blocks == 8u ? 124u : 100u) && strips * (blocks + 9u) <= 3300u) return true;
    if (bands == 7u && blocks >= 9u && blocks <= 17u && strips <= 119u) return true;
    if (blocks >= 48u && (bands >= 13u || (bands >= 8u && strips >= 96u))) return true;
    return (blocks >= (bands > 2u ? 68u : 100u) && (bands >= 6u || all > 560u)) || (blocks >= 110u && all > 420u);
}

}  // namespace pilc
